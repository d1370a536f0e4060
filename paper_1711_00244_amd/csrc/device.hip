// gfx950 kernels and their launchers: record-parallel Huffman decode, position
// prefix sums, codebook lookup, and the fused sparse-weight x dense-activation
// product (Algorithm 2 of the paper, re-cast for 64-lane wavefronts).
//
// One wavefront owns one chunk: up to 64 lane records of 64 bits, all of one block.
// Lane l reads record l with one 64-bit load (a full 512-byte burst per wavefront).
// A record holds n entries: their value-index codewords run up from bit 4, their
// relative-index codewords run down from bit 63, so a lane decodes both spans side
// by side from two shift registers with two decode tables held in LDS.
//   decode  both spans, entry by entry, symbols kept in registers, z + 1 summed per lane
//   scan    one wavefront prefix sum turns lane sums into each lane's starting
//           position (Algorithm 1 step 7) and lane counts into output slots
//   use     the entries in order, each with its position: store it (decode_layer),
//           multiply-accumulate it (sparse forward) or place it in a dense tile (MFMA forward)
//
// One translation unit: this file holds the host side (device image of a layer, launch
// shapes, the entry points) and includes the kernels - decode.hpp (wavefront primitives,
// decoding and placement passes), sparse_kernels.hpp, mfma_kernels.hpp, wide_kernels.hpp, rows_kernels.hpp, bf16_kernels.hpp,
// conv_kernels.hpp, conv_plane_kernels.hpp, finish_kernels.hpp, layer_kernels.hpp.
#include <hip/hip_runtime.h>
#include <type_traits>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <memory>
#include <vector>

#include "layer.hpp"

namespace cl {

#define HIP_TRY(expr)                                                                         \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess) return fail(CL_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

// A launch of n workgroups along x; more than a grid holds is refused, not wrapped.
#define GRID_TRY(g, n)                                                                        \
    do {                                                                                      \
        const int64_t n_ = (n);                                                               \
        if (n_ < 1 || n_ > INT32_MAX) return fail(CL_EUNSUPPORTED, "a launch of %lld workgroups does not fit a grid", (long long)n_); \
        (g) = dim3((unsigned)n_);                                                             \
    } while (0)

constexpr int kWaves = 8;                 // wavefronts per workgroup
constexpr int kSparseChunksPerWave = 1;   // chunks a wavefront of the sparse kernel decodes, one after the other
                                          // (2 amortises the table copy but measured 18 % slower at batch 1)
constexpr int kThreads = kWaves * 64;

// Everything a kernel needs to read a layer, passed by value.
struct LayerDev {
    const uint64_t *records;
    const cl_chunk_meta *meta;
    const uint32_t *panel_chunk;
    const uint32_t *block_chunk;
    const ChunkSlot *slot;               // may be null, as row_ptr (cl_layer::slot)
    const uint32_t *chunk_half;          // null unless the blocks are at most 128 x 128 (with group_ptr)
    const uint32_t *group_ptr;
    const uint16_t *row_ptr;
    const void *rec_pos;                 // null unless the small-batch kernel's wavefronts have tiles of their own
    const float *codebook;
    const uint4 *tables;                 // both decode tables and the codebook as they lie in LDS (carve)
    int M, K, bh, bw, nbw;
    int val_bits, idx_bits, ncode;       // index widths of the decode tables, codebook entries
    int pos32;                           // rec_pos has 32 bits a record, not 16
    int block_slots, row_ptrs;           // slots of a block in `slot`, entries of a block in row_ptr
    int table_rows;                      // 16-byte rows of the table image (tables + codebook)
    uint32_t n_chunks;
    int panel0;                          // first block row of a launch that covers only some (a filter group); else 0
};

// Bytes of the table image: both decode tables - the larger one first, so that each starts at
// a multiple of its size - then the codebook, each padded to 16 bytes.
static size_t table_image_bytes(int vbits, int ibits, int ncode)
{
    const size_t tb = (((size_t)1 << vbits) + ((size_t)1 << ibits)) * sizeof(lut_t);
    return ((tb + 15) & ~(size_t)15) + (((size_t)ncode * 4 + 15) & ~(size_t)15);
}

static LayerDev make_dev(const cl_layer *L)
{
    LayerDev d;
    d.records = L->dev.records;
    d.meta = L->dev.meta;
    d.panel_chunk = L->dev.panel_chunk;
    d.block_chunk = L->dev.block_chunk;
    d.slot = L->dev.slot;
    d.block_slots = L->block_slots;
    d.row_ptrs = L->row_ptrs;
    d.chunk_half = L->dev.chunk_half;
    d.group_ptr = L->dev.group_ptr;
    d.codebook = L->dev.codebook;
    d.row_ptr = L->dev.row_ptr;
    d.rec_pos = L->dev.rec_pos;
    d.pos32 = L->rec_pos32.empty() ? 0 : 1;
    d.tables = (const uint4 *)L->dev.tables;
    d.M = L->desc.M;
    d.K = L->desc.K;
    d.bh = L->desc.block_h;
    d.bw = L->desc.block_w;
    d.nbw = L->nbw;
    d.val_bits = L->val_lut_bits;
    d.idx_bits = L->idx_lut_bits;
    d.ncode = 1 << L->desc.weight_bits;
    d.table_rows = (int)(table_image_bytes(L->val_lut_bits, L->idx_lut_bits, d.ncode) / 16);
    d.n_chunks = (uint32_t)L->n_chunks;
    d.panel0 = 0;
    return d;
}

#include "decode.hpp"
#include "sparse_kernels.hpp"
#include "mfma_kernels.hpp"
#include "wide_kernels.hpp"
#include "rows_kernels.hpp"
#include "bf16_kernels.hpp"
#include "conv_kernels.hpp"
#include "conv_plane_kernels.hpp"
#include "finish_kernels.hpp"
#include "layer_kernels.hpp"

// ------------------------------------------------------------------------- //
// host side
// ------------------------------------------------------------------------- //
struct DeviceLimits {
    int device = -1;
    int cus = 0;
    size_t max_lds = 0;
};

static int32_t device_limits(DeviceLimits &dl)
{
    static thread_local DeviceLimits cache;
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (cache.device != dev) {
        int cus = 0, lds = 0;
        HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        HIP_TRY(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
        cache.device = dev;
        cache.cus = cus;
        cache.max_lds = (size_t)lds;
    }
    dl = cache;
    return CL_OK;
}

// Raises a kernel's dynamic LDS limit when a launch needs more than any before it on
// this device (the attribute sticks; asking again for every launch costs a runtime
// call each time).  `seen` belongs to one kernel instantiation.
constexpr int kMaxDevices = 64;
struct LdsLimit { std::atomic<size_t> bytes[kMaxDevices]; };

static int32_t ensure_lds(const void *kernel, size_t lds, LdsLimit &seen)
{
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    const bool tracked = dev >= 0 && dev < kMaxDevices;
    if (tracked && seen.bytes[dev].load(std::memory_order_relaxed) >= lds) return CL_OK;
    HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    if (tracked) seen.bytes[dev].store(lds, std::memory_order_relaxed);
    return CL_OK;
}

// Event bracket around the main kernel of the last forward call (benchmarks only).
struct KernelTiming {
    bool on = false, valid = false;
    hipEvent_t a = nullptr, b = nullptr;
    int launches = 0;
};
static KernelTiming g_timing;

static void timing_begin(hipStream_t st)
{
    if (!g_timing.on) return;
    g_timing.launches = 0;
    g_timing.valid = hipEventRecord(g_timing.a, st) == hipSuccess;
}

static void timing_end(hipStream_t st, int launches)
{
    if (!g_timing.on || !g_timing.valid) return;
    g_timing.launches = launches;
    g_timing.valid = hipEventRecord(g_timing.b, st) == hipSuccess;
}

// Scratch for the entry point that may not allocate: one array per GPU, placed by the
// loader, held until the process ends.  In host code the array's name is only a handle
// for hipGetSymbolAddress; kernels get the address that call returns for the current
// device.
static __device__ __align__(256) unsigned char g_static_scratch[CL_STATIC_SCRATCH_BYTES];

constexpr int kMaxScratchDevices = 64;
static std::atomic<void *> g_static_scratch_ptr[kMaxScratchDevices];

// Address of the current device's copy of the scratch array (looked up once per device).
static int32_t static_scratch(void **out)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxScratchDevices) return fail(CL_EUNSUPPORTED, "device %d: static scratch is tracked for devices 0..%d", dev, kMaxScratchDevices - 1);
    void *p = g_static_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch)));
        if (!p) return fail(CL_EHIP, "hipGetSymbolAddress gave a null address");
        g_static_scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return CL_OK;
}

void release_device(cl_layer *L)
{
    if (L->dev.blob) {
        (void)hipFree(L->dev.blob);
        L->dev = DeviceImage{};
    }
}

static int32_t require_device(const cl_layer *L)
{
    if (!L) return fail(CL_EINVAL, "null layer");
    if (!L->dev.blob) return fail(CL_EINVAL, "layer is not on the device: call cl_layer_upload first");
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != L->dev.device) return fail(CL_EINVAL, "layer was uploaded to device %d, current device is %d", L->dev.device, dev);
    return CL_OK;
}

}  // namespace cl

using namespace cl;

extern "C" int32_t cl_layer_upload(cl_layer *L)
try {
    if (!L) return fail(CL_EINVAL, "null layer");
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) return fail(CL_EHIP, "no HIP device");
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (L->dev.blob && L->dev.device == dev) return CL_OK;
    {
        // set-up time: find this device's copy of the static scratch array now, so that the
        // non-allocating entry point has nothing left to look up (a device beyond the
        // tracked range is refused there, not here)
        void *scratch = nullptr;
        if (dev >= 0 && dev < kMaxScratchDevices)
            if (int32_t rc = static_scratch(&scratch)) return rc;
    }
    release_device(L);
    struct Sec { const void *src; size_t bytes; size_t off; };
    // decode tables + codebook, laid out as in LDS
    const int ncode = 1 << L->desc.weight_bits;
    std::vector<char> image(table_image_bytes(L->val_lut_bits, L->idx_lut_bits, ncode), 0);
    {
        const size_t vb = L->val_lut.size() * sizeof(lut_t), ib = L->idx_lut.size() * sizeof(lut_t);
        const bool values_first = vb >= ib;
        std::memcpy(image.data() + (values_first ? 0 : ib), L->val_lut.data(), vb);
        std::memcpy(image.data() + (values_first ? vb : 0), L->idx_lut.data(), ib);
        std::memcpy(image.data() + ((vb + ib + 15) & ~(size_t)15), L->codebook.data(), L->codebook.size() * 4);
    }
    Sec secs[12] = {
        {L->records.data(), L->records.size() * 8, 0},
        {L->meta.data(), L->meta.size() * sizeof(cl_chunk_meta), 0},
        {L->block_ptr.data(), L->block_ptr.size() * 4, 0},
        {L->panel_chunk.data(), L->panel_chunk.size() * 4, 0},
        {image.data(), image.size(), 0},
        {L->block_chunk.data(), L->block_chunk.size() * 4, 0},
        {L->slot.data(), L->slot.size() * sizeof(ChunkSlot), 0},
        {L->chunk_half.data(), L->chunk_half.size() * 4, 0},
        {L->group_ptr.data(), L->group_ptr.size() * 4, 0},
        {L->row_ptr.data(), L->row_ptr.size() * 2, 0},
        {L->rec_pos16.data(), L->rec_pos16.size() * 2, 0},
        {L->rec_pos32.data(), L->rec_pos32.size() * 4, 0},
    };
    size_t total = 0;
    for (auto &s : secs) { s.off = total; total += (s.bytes + 255) / 256 * 256; }
    total += 256;
    // The small sections travel together, with zeros between them; a section of 1 MB and more goes by itself from where it lies
    // (what lies behind it up to the next one is read by nobody).  The AlexNet-shaped fc6, 7 MB: 430 us, 560 with all of
    // them put together first in new memory.
    constexpr size_t kOwnCopy = 1 << 20;
    std::vector<char> together;
    struct Copy { size_t off; const void *src; size_t bytes; };
    std::vector<Copy> copies;
    size_t end = 0;                                     // of what is put together, from its first byte on the device
    size_t small = 0;
    for (const auto &s : secs) small += s.bytes < kOwnCopy ? (s.bytes + 255) / 256 * 256 : 0;
    together.assign(small + 256, 0);
    for (size_t i = 0; i < std::size(secs); ++i) {
        const auto &s = secs[i];
        if (s.bytes >= kOwnCopy) {
            copies.push_back({s.off, s.src, s.bytes});
            continue;
        }
        const bool joins = i > 0 && secs[i - 1].bytes < kOwnCopy;
        const size_t padded = (i + 1 < std::size(secs) ? secs[i + 1].off : total) - s.off;
        if (!joins) copies.push_back({s.off, together.data() + end, 0});
        if (s.bytes) std::memcpy(together.data() + end, s.src, s.bytes);
        end += padded;
        copies.back().bytes += padded;
    }
    char *blob = nullptr;
    if (hipMalloc((void **)&blob, total) != hipSuccess) return fail(CL_ENOMEM, "hipMalloc of %zu bytes failed", total);
    for (const Copy &c : copies)
        if (c.bytes && hipMemcpy(blob + c.off, c.src, c.bytes, hipMemcpyHostToDevice) != hipSuccess) {
            (void)hipFree(blob);
            return fail(CL_EHIP, "hipMemcpy to device failed");
        }
    L->dev.device = dev;
    L->dev.blob = blob;
    L->dev.blob_bytes = total;
    L->dev.records = (const uint64_t *)(blob + secs[0].off);
    L->dev.meta = (const cl_chunk_meta *)(blob + secs[1].off);
    L->dev.block_ptr = (const uint32_t *)(blob + secs[2].off);
    L->dev.panel_chunk = (const uint32_t *)(blob + secs[3].off);
    L->dev.block_chunk = (const uint32_t *)(blob + secs[5].off);
    L->dev.slot = L->slot.empty() ? nullptr : (const ChunkSlot *)(blob + secs[6].off);
    L->dev.chunk_half = L->group_ptr.empty() ? nullptr : (const uint32_t *)(blob + secs[7].off);
    L->dev.group_ptr = L->group_ptr.empty() ? nullptr : (const uint32_t *)(blob + secs[8].off);
    L->dev.row_ptr = L->row_ptr.empty() ? nullptr : (const uint16_t *)(blob + secs[9].off);
    L->dev.rec_pos = !L->rec_pos16.empty() ? blob + secs[10].off : !L->rec_pos32.empty() ? blob + secs[11].off : nullptr;
    L->dev.tables = blob + secs[4].off;
    L->dev.codebook = (const float *)(blob + secs[4].off + ((L->val_lut.size() + L->idx_lut.size()) * sizeof(lut_t) + 15) / 16 * 16);
    clear_error();
    return CL_OK;
} catch (...) {
    return fail_with_exception();
}

// decode_blocks_kernel takes a few thousand cycles for a block, most of them latencies, however small
// the block is.  With blocks of less than 64 x 64 the chunk kernel, which has a wavefront for
// each, is faster in spite of the second pass over the dense matrix (4096 x 4096: blocks of
// 32 x 32, 31 and 53 us; of 64 x 64, 31 and 21 us), and where no dense matrix is asked for it
// already is with somewhat larger ones (4096 x 25088: blocks of 64 x 64, 30 and 70 us; of
// 128 x 128, 28 and 25 us).
static bool decode_by_blocks(const cl_layer *L, bool dense)
{
    return !L->slot.empty() && (int64_t)L->desc.block_h * L->desc.block_w >= (dense ? 64 * 64 : 96 * 96);
}

extern "C" int32_t cl_decode_layer(const cl_layer *L, uint8_t *d_val_sym, uint8_t *d_idx_sym,
                                   uint32_t *d_block_ptr, float *d_dense, void *stream)
{
    if (int32_t rc = require_device(L)) return rc;
    hipStream_t st = (hipStream_t)stream;
    const LayerDev D = make_dev(L);
    if (decode_by_blocks(L, d_dense != nullptr) && (d_val_sym || d_idx_sym || d_block_ptr || d_dense)) {
        DeviceLimits dl;
        if (int32_t rc = device_limits(dl)) return rc;
        const int stage = ((int)L->max_block_entries + 31) / 16 * 16;           // (and up to 15 bytes before the first)
        const size_t lds = smem_fixed_bytes(D.val_bits, D.idx_bits, D.ncode) + kDecodeTile + 2 * (size_t)stage;
        static LdsLimit seen;
        if (int32_t rc = ensure_lds((const void *)decode_blocks_kernel, lds, seen)) return rc;
        // as many workgroups as are resident at once, each with the same number of blocks where
        // that divides
        const int64_t resident = (int64_t)dl.cus * std::max<int64_t>(1, std::min<int64_t>(8, dl.max_lds / lds));
        const int64_t each = (L->n_blocks + resident - 1) / resident;
        hipLaunchKernelGGL(decode_blocks_kernel, dim3((unsigned)((L->n_blocks + each - 1) / each)), dim3(kDecodeThreads), lds, st, D, L->dev.block_ptr,
                           (int)L->n_blocks, d_val_sym, d_idx_sym, d_block_ptr, d_dense, stage);
        HIP_TRY(hipGetLastError());
        clear_error();
        return CL_OK;
    }
    if (d_block_ptr)
        HIP_TRY(hipMemcpyAsync(d_block_ptr, L->dev.block_ptr, (size_t)(L->n_blocks + 1) * 4, hipMemcpyDeviceToDevice, st));
    if (d_dense) {
        const size_t n = (size_t)L->desc.M * L->desc.K;
        hipLaunchKernelGGL(fill_kernel, dim3((unsigned)std::min<size_t>((n + 255) / 256, 4096)), dim3(256), 0, st, d_dense, n, 0.0f);
        HIP_TRY(hipGetLastError());
    }
    if (L->n_chunks > 0 && (d_val_sym || d_idx_sym || d_dense)) {
        const size_t lds = smem_fixed_bytes(D.val_bits, D.idx_bits, D.ncode);
        const dim3 grid((unsigned)((L->n_chunks + kWaves - 1) / kWaves));
        hipLaunchKernelGGL(decode_kernel, grid, dim3(kThreads), lds, st, D, d_val_sym, d_idx_sym, d_dense);
        HIP_TRY(hipGetLastError());
    }
    clear_error();
    return CL_OK;
}

namespace {

// Most columns (images, or images x output pixels) of one dense-tile launch: keeps the
// kernels' 32-bit column arithmetic and the y extent of the layout kernels' grids in range.
constexpr int kMaxTileColumns = 1 << 21;

// Launch shape of fc_rows_kernel, the sparse path's kernel for more than a few images.
struct RowsPlan {
    int ipl = 0;             // images per lane (0: the kernel is not used)
    int group = 1;           // blocks decoded and multiplied at a time
    int run = 0;             // images per launch: whole image tiles, or all there are
    int splits = 1;          // workgroups sharing the blocks of one block row
    int list_cap = 0;        // entries a block's list has room for
    int64_t cost = 0;        // modelled cycles of the launches (same units as mfma_shape's)
    size_t lds = 0, part_bytes = 0;
    int padded(int images) const { return (images + 16 * ipl - 1) / (16 * ipl) * (16 * ipl); }
};

// At one image a layer of more block rows than this stays on two launches where eight wavefronts have all chunks of a block
// row: eight of fc_sparse_whole_kernel's sixteen and more clear, stage and wait for the others, which the launch it saves
// (2 us) pays for up to some 2.9 k block rows of one chunk and 4.1 k of eight.  (us a call, one launch / two: one chunk, 2048
// block rows 13.8 / 14.4, 3072 19.6 / 19.1, 4096 25.6 / 24.1, 65536 424 / 346; four chunks 20.7 / 20.8 at 3072, 26.6 / 25.9 at
// 4096; eight 23.1 / 24.1, 29.7 / 30.3, 122 / 112 at 16384; nine, two workgroups of eight wavefronts, 131 / 190 there.
// Two images, one chunk: 15.5 / 18.9, 28.9 / 34.1 and 488 / 501; four images 497 / 817.)
int64_t whole_narrow_rows(int64_t chunks) { return 2816 + 160 * chunks; }

// GPU time of fc_sparse_whole_kernel less that of the two launches, in ns, where a wavefront has more than one chunk to take
// (up to one, sixteen to a block row, the one launch is 1 to 4 us shorter everywhere).  A wavefront's chunks come one after the
// other, each as long as its longest record, which the entries of a record stand for, twice as long where a position takes a
// division to split; all columns are staged.  `full`: the two launches have so many workgroups to a CU, one and a half and more, that
// they take longer themselves.  Fitted to thirteen shapes of block and density, 4 to 48 chunks, 1 to 300 block rows (rms 0.6 us).  At one image,
// us on the GPU, one launch / two: 1024 rows at 10 %, 40 chunks 8.5 / 7.1, 20 chunks 6.0 / 6.9; blocks 128 x 128 at
// 1.8 %, fourteen entries to a record, 24 chunks 8.1 / 8.0, 48 chunks 12.5 / 7.8.
int64_t whole_extra(const cl_layer *L, int bt, bool full)
{
    const int64_t chunks = L->max_panel_chunks, K = L->desc.K, wide = (L->desc.block_w & (L->desc.block_w - 1)) ? 2 : 1;
    const int64_t steps = L->entries * 10 * wide / std::max<int64_t>(1, L->n_records);           // tenths
    if (bt > 2) return full ? INT64_MIN : chunks * (77 + steps * 8 / 10) - 3730;
    if (bt == 2) return full ? chunks * (41 + steps * 66 / 100) + K / 4 - 3790 : chunks * (105 + steps * 68 / 100) + K / 3 - 4200;
    return full ? chunks * (28 + steps * 74 / 100) + K / 7 - 3390 : chunks * (107 + steps * 48 / 100) + K / 7 - 3840;
}

// Up to this whole_extra (within the fit's error of none) one launch is the faster one whatever waits for it.  A call of one
// launch by itself also spares the host a launch, 2.4 us, which bounds calls one behind the other (1024 x 1024 at 10 %: 11.7 -> 9.1 us); one
// that is waited for has only some of that, since the host makes the second launch beside the first (23.7 -> 24.3 us; 20 chunks 23.5 -> 21.9): up
// to the second figure the first gains more than the second loses.
constexpr int64_t kWholeExtra = 200, kWholeExtraAlone = 2300;

// Launch shape of the sparse forward path for one layer and batch.
struct SparsePlan {
    RowsPlan rows;           // the launch, if fc_rows_kernel takes it; else:
    int bt_max = 1;          // batch tile of the main kernel (power of two, <= 16)
    int wg_per_panel = 0;    // workgroups per block row (8 wavefronts of kSparseChunksPerWave chunks each)
    int xwant = 0;           // activation columns to stage in LDS per image (3 blocks wide)
    size_t fixed = 0;        // LDS bytes of tables + codebook
    size_t part_bytes = 0;   // partial-tile buffer in the workspace
    int cus = 1;
    // LDS of fc_sparse_whole_kernel, 0 where it does not take the layer (a block row of more chunks than it has places, no tile
    // per chunk, more than a workgroup's 64 KiB, more threads than a launch may have: its workgroups have twice those of the
    // two launches, which at one image take up to twice as many block rows; where two launches are the faster ones).  alone(): the
    // call is this launch, made by the host as it goes.
    template <class Alone> size_t whole_lds(const cl_layer *L, int bt, Alone alone) const
    {
        if (bt > kWholeBT || !private_tiles(L->desc.block_h, bt) || L->max_panel_chunks > kWholeWaves * kWholeRounds) return 0;
        if ((uint64_t)L->n_panels * (kWholeWaves * 64) > UINT32_MAX) return 0;
        if (bt == 1 && wg_per_panel == 1 && L->n_panels > whole_narrow_rows(L->max_panel_chunks)) return 0;
        const size_t lds = fixed + ((size_t)wg_per_panel * kWaves * L->desc.block_h + L->desc.K) * 4 * bt;
        if (lds > 64 * 1024) return 0;
        if (L->max_panel_chunks > kWholeWaves && whole_extra(L, bt, 2 * (int64_t)L->n_panels * wg_per_panel > 3 * (int64_t)cus) > kWholeExtra &&
            (whole_extra(L, bt, false) > kWholeExtraAlone || !alone())) return 0;
        return lds;
    }
    int xcap_for(int bt) const { return (size_t)xwant * 4 * bt <= 32 * 1024 ? xwant : 0; }
    size_t lds_for(const cl_layer *L, int bt) const
    {
        const size_t tiles = private_tiles(L->desc.block_h, bt) ? kWaves : 1;
        return fixed + (tiles * L->desc.block_h + xcap_for(bt)) * 4 * bt;
    }
};

bool mfma_capable(const cl_layer *L) { return L->desc.block_h <= kTile && L->desc.block_w <= kTile; }

// From this many images on the sparse path runs fc_rows_kernel where the layer's blocks allow
// (fc6 / fc7 / fc8 of the AlexNet-shaped stack, us a call: 24 / 16 / 14 at 8 images on the small-batch
// kernel, 28 / 17 / 18 on this one; at 9-16 images, two launches there, 44 / 30 / 25).
constexpr int kRowsBatch = 9;

// It pays a fixed part per block (some 3 k cycles), the small-batch kernel one per chunk (under 1 k for
// eight images).  So where a block is one chunk and every CU has many, up to 16 images - two launches
// there - are faster on the small-batch kernel (4096 x 4096 at 9 %, us a call at 9 / 16 images, this kernel
// and the small-batch one: blocks of 16 x 16 323 / 349 and 151 / 213; 32 x 32 89 / 95 and 54 / 71; 16 x 128
// 51 / 53 and 40 / 54; 64 x 64 33 / 34 and 37 / 49.  32 images: 32 x 32 112 and 140, 16 x 128 62 and 106.
// 1000 x 4096 at 25 %, 8 blocks to a CU, 16 x 128: 24 / 24 and 29 / 37; 16 to a CU, 32 x 32: 32 / 33 and 26 / 32.)
constexpr int kRowsCells = 64 * 64, kRowsBlocksPerCu = 12;

bool rows_kernel_pays(const cl_layer *L, int batch, int cus)
{
    if (batch < kRowsBatch) return false;
    return batch > 16 || (int64_t)L->desc.block_h * L->desc.block_w >= kRowsCells || L->n_blocks <= (int64_t)kRowsBlocksPerCu * std::max(1, cus);
}

// Most scratch fc_rows_kernel takes for its partial tiles, whatever the batch: what the entry point
// without a workspace has.  A batch whose tiles, unsplit, take more is cut into runs, one launch after
// the other.  (A tile of 64 images is 32 KiB, so two per CU fit: a run of that size keeps the chip
// busy.)
constexpr size_t kRowsScratch = CL_STATIC_SCRATCH_BYTES;

// Launch shape of fc_rows_kernel; false where it does not fit (blocks above 128 x 128, a layer
// without the tables it reads, more weights in a block than its list has room for in LDS, so many
// block rows that a tile of sixteen images of each exceeds kRowsScratch).
bool plan_rows(const cl_layer *L, int batch, const DeviceLimits &dl, RowsPlan &P)
{
    if (L->row_ptr.empty() || batch > kMaxTileColumns) return false;
    const size_t image_bytes = (size_t)L->n_panels * kTile * sizeof(float);       // of the partial tiles, unsplit
    const int64_t most = (int64_t)(kRowsScratch / image_bytes);
    if (most < 16) return false;
    P.ipl = batch <= 16 || most < 32 ? 1 : batch <= 32 || most < 64 ? 2 : 4;
    const int images = 16 * P.ipl;
    const int runs = (int)((batch + most / images * images - 1) / (most / images * images));
    P.run = runs == 1 ? batch : P.padded((batch + runs - 1) / runs);
    const int Bp = P.padded(P.run);
    P.list_cap = (int)((L->max_block_nnz + kListSlack + 7) / 8 * 8);
    const size_t tables = table_image_bytes(L->val_lut_bits, L->idx_lut_bits, 1 << L->desc.weight_bits);
    auto lds_of = [&](int group) { return tables + 2 * (size_t)group * (images * kXsColumns * sizeof(float) + P.list_cap * sizeof(uint16_t)); };
    if (lds_of(1) > dl.max_lds) { P.ipl = 0; return false; }
    // Blocks to a group and split of the block rows, as on the other paths, in cycles per
    // workgroup: a start; per group of blocks a part that does not depend on what is in it
    // (latencies, the barrier), per block and per surviving weight; the partial tiles.  Fitted to
    // the AlexNet- and VGG-shaped fc6 / fc7 / fc8 at 16, 32 and 64 images, when a group's turn still waited for its loads.  It does
    // not any more, and all parts have become shorter alike: over 1400 calls (a hundred layers drawn from 200 x 500 to 8192 x
    // 25088, densities of 3 to 40 %, 12 to 512 images) a call takes 0.83 of its price, rms 7.7 %, and with every constant fitted
    // anew 7.2 %.  Groups and splits come out the same either way (AlexNet-shaped fc6, us a call: 24.4, 28.2 and 40.7; one block
    // to a group 30.0, 32.2 and 40.7 - at 16 images before four lanes had a row); against the other paths the price is too high, which kAutoLaunch makes up for in part.
    // With 16 images (four lanes to a row, groups of one, two or four blocks) its parts are those of 4096-row layers of 4096 to 25088 columns
    // and 3 to 30 %, to the same 0.83.  It holds for other heights: of 281 calls at 9 to 16 images drawn from 96 to 8192 rows, 128 to 25088 columns and 2 to
    // 40 % none is slower than with two rows to a quarter wavefront and that form's price (1.007 times at most), 0.96 times on average.
    static const struct { int groups, group, block, weight_x20; } kFit[3] = {{4, 4400, 630, 29}, {3, 2200, 3000, 34}, {1, 2200, 3900, 51}};
    const auto &fit = kFit[P.ipl / 2];
    const int64_t tiles = (int64_t)L->n_panels * (Bp / images);
    const int cus = std::max(1, dl.cus);
    const int64_t nnz_block = L->n_blocks ? L->nnz / L->n_blocks : 0;
    const int64_t per_block = fit.block + nnz_block * fit.weight_x20 / 20, per_group = fit.group, start = 12000;
    const int sp_max = (int)std::max<int64_t>(1, std::min<int64_t>({L->nbw, (3 * (int64_t)cus + tiles - 1) / tiles, (int64_t)(kRowsScratch / (image_bytes * Bp))}));
    int64_t best = -1;
    for (int group = 1; group <= fit.groups && lds_of(group) <= dl.max_lds; group += P.ipl == 1 ? group : 1)
        for (int sp = 1; sp <= sp_max; ++sp) {
            const int64_t rounds = (tiles * sp + cus - 1) / cus, blocks = (L->nbw + sp - 1) / sp;
            const int64_t t = rounds * (start + (blocks + group - 1) / group * per_group + blocks * per_block) +
                              (int64_t)image_bytes * sp * Bp * 3 / 4000;
            if (best < 0 || t < best) {
                best = t;
                P.splits = sp;
                P.group = group;
            }
        }
    P.lds = lds_of(P.group);
    P.cost = best * runs;
    P.part_bytes = image_bytes * P.splits * Bp;
    return true;
}

// (one_tile: the caller wants the whole batch, up to 16 images, in one batch tile; rows: the launch shape
// of fc_rows_kernel where the caller has it already)
int32_t plan_sparse(const cl_layer *L, int batch, const DeviceLimits &dl, SparsePlan &P, bool one_tile = false, const RowsPlan *rows = nullptr)
{
    const size_t max_lds = dl.max_lds;
    if (!one_tile && rows_kernel_pays(L, batch, dl.cus)) {
        if (rows) P.rows = *rows;
        if (rows || plan_rows(L, batch, dl, P.rows)) {
            P.part_bytes = P.rows.part_bytes;
            return CL_OK;
        }
    }
    P.cus = std::max(1, dl.cus);
    P.fixed = table_image_bytes(L->val_lut_bits, L->idx_lut_bits, 1 << L->desc.weight_bits);
    P.xwant = (int)std::min<int64_t>(L->desc.K, (1 + 2 * kSparseChunksPerWave) * (int64_t)L->desc.block_w);
    // largest power-of-two batch tile (<= 16) that fits; prefer to stay under 64 KiB
    size_t budget = std::min<size_t>(max_lds, 64 * 1024);
    if (P.lds_for(L, 1) > budget) budget = max_lds;
    if (P.lds_for(L, 1) > budget) return fail(CL_EUNSUPPORTED, "block_h %d needs more LDS than a workgroup has", L->desc.block_h);
    // two launches with a tile per wavefront are faster than one of 16 images through atomics
    P.bt_max = !one_tile && private_tiles(L->desc.block_h, kPrivateTileBT) ? kPrivateTileBT : 16;
    while (P.bt_max > 1 && (P.lds_for(L, P.bt_max) > budget || P.bt_max / 2 >= batch)) P.bt_max >>= 1;
    P.wg_per_panel = (int)((L->max_panel_chunks + kWaves * kSparseChunksPerWave - 1) / (kWaves * kSparseChunksPerWave));
    P.part_bytes = (size_t)L->n_panels * P.wg_per_panel * L->desc.block_h * P.bt_max * sizeof(float);
    return CL_OK;
}

// Whether a stack could leave out the finishing kernel between two layers on this path,
// as far as this layer goes (as producer or consumer): the batch is a single batch tile,
// so that there is one set of partial tiles, and - for the consumer - every workgroup
// stages its activation columns in LDS, where the sum of the tiles is formed.
bool sparse_can_fold(const cl_layer *L, const SparsePlan &P, int batch)
{
    if (P.rows.ipl || batch > P.bt_max || (batch & (batch - 1))) return false;
    const int64_t widest = std::min<int64_t>(L->desc.K, (int64_t)L->max_group_blocks * L->desc.block_w);
    return widest <= P.xcap_for(batch);
}

// Launch shape of the MFMA path.
struct MfmaPlan {
    int nq = 4;              // 32-image groups per workgroup tile
    bool bf16 = false;       // three bf16 products instead of one fp32 product
    int Bp = 0;              // batch rounded up to whole image tiles
    int splits = 1;          // workgroups sharing the blocks of one block row
    size_t lds = 0;
    size_t xt_bytes = 0, part_bytes = 0;
};

// columns per workgroup of the finishing kernel: as many as leave 1024 workgroups
int reduce_col_tile(int panels, int ncols)
{
    int ct = kColTile;
    while (ct > 1 && (int64_t)panels * ((ncols + ct - 1) / ct) < 1024) ct >>= 1;
    return ct;
}

// rows of the block-by-block activation layout, tail included
size_t xt_rows(const cl_layer *L) { return (size_t)L->nbw * kTile + kXtTailRows; }

// Image tile, padded column count and split of the block rows for `ncols` columns and
// `panels` block rows, from a small model of a layer's launches with measured constants
// (cycles per workgroup: 12 k to start; per block 5 k of decoding and bookkeeping plus
// 4.1 k of multiplies per 32 columns of the tile - 1.5 k on the bf16 matrix cores;
// workgroups run in rounds of one per CU; and 3 cycles per 4 KB of partial tiles, which
// are written, flushed at the kernel's end and read again by the finishing kernel -
// 2 per 5 KB next to the gathered convolution's kernel, nothing where one workgroup per
// block row writes the output itself, `direct`).  Fitted
// to sweeps over every tile width and split of the AlexNet and VGG-16 FC layers at 8 to
// 1024 images: the choice is the fastest measured shape for the large layers and
// within 3 % of it on average for a 1000-row layer, where the partial tiles decide.  (The bf16 kernel has become faster
// since, its wide tiles most: over the calls of plan_rows a thousand cycles of price take 0.37 us with 32 and 64 columns to a
// tile, 0.30 with 128 and 0.23 with 256.  Its price has not been fitted again.)  The
// gathered convolution's kernel is priced at 13 k cycles a block (two phases), 7.5 k with blocks of at most 64
// rows or two terms, and 4 k for an item; against its predecessor's price (8 k and 17.9 k for any block) 0 to
// 4 % faster over forty convolutions, none slower by more than 1 %.  (Fitted with six products of the terms; with
// eight a block takes about 14.5 k, a price that gives thirty-two convolutions the same splits.)
void mfma_shape(const cl_layer *L, int panels, int ncols, int cus, bool bf16, int &nq, int &np, int &splits, bool gathered = false,
                bool direct = false, int64_t *cost = nullptr)
{
    cus = std::max(1, cus);
    nq = 0;
    int64_t best = -1;
    for (int q : {1, 2, 4, 8}) {
        if (gathered && 32 * q != kConvColumns) continue;      // conv_mfma_kernel has one tile width
        const int w = 32 * q;
        const int cols = (ncols + w - 1) / w * w;
        const int64_t tiles = (int64_t)panels * (cols / w);
        // any split up to three rounds of workgroups (eight for the gathered convolution,
        // whose long block rows gain from them): more, shorter workgroups can beat one
        // round that leaves CUs idle
        const int64_t max_rounds = gathered ? 8 : 3;
        const int sp_max = (int)std::max<int64_t>(1, std::min<int64_t>(L->nbw, (max_rounds * cus + tiles - 1) / tiles));
        for (int sp = 1; sp <= sp_max; ++sp) {
            const int64_t rounds = (tiles * sp + cus - 1) / cus;
            const int64_t blocks = (L->nbw + sp - 1) / sp;
            // blocks decoded beforehand; a workgroup that goes on to its next item starts quickly
            int64_t t = gathered ? rounds * (4000 + blocks * (bf16 || L->desc.block_h <= 64 ? 7500 : 13000))
                              : rounds * (12000 + blocks * (5000 + (bf16 ? 1500 : 4100) * q));
            if (!(direct && sp == 1)) t += (int64_t)panels * sp * cols * L->desc.block_h * (int64_t)sizeof(float) * (gathered ? 2 : 3) / (gathered ? 5000 : 4000);
            if (best < 0 || t < best) {
                best = t;
                nq = q;
                np = cols;
                splits = sp;
            }
        }
    }
    if (cost) *cost = best;
}

size_t mfma_lds_bytes(const cl_layer *L, bool bf16)
{
    const size_t tables = table_image_bytes(L->val_lut_bits, L->idx_lut_bits, 1 << L->desc.weight_bits);
    return bf16 ? tables + 2 * (size_t)kBf16BufFloats * 4 + ((size_t)4 << L->desc.weight_bits) : tables + 2 * (size_t)kWTileBytes;
}

// bf16 elements of one plane of the split activations, read-ahead tail included
size_t xb_plane_elems(const cl_layer *L, int np) { return ((size_t)L->nbw * 8 + kXbTailGroups) * np * 16; }

// bytes of the activations as the dense-tile kernel of the given precision reads them
size_t xt_bytes_for(const cl_layer *L, int np, bool bf16)
{
    const size_t raw = bf16 ? 2 * xb_plane_elems(L, np) * sizeof(uint16_t) : xt_rows(L) * np * sizeof(float);
    return (raw + 255) / 256 * 256;
}

int32_t plan_mfma(const cl_layer *L, int batch, bool bf16, const DeviceLimits &dl, MfmaPlan &P)
{
    if (!mfma_capable(L)) return fail(CL_EUNSUPPORTED, "the MFMA path needs blocks of at most %d x %d", kTile, kTile);
    if (batch > kMaxTileColumns) return fail(CL_EUNSUPPORTED, "the dense-tile paths take at most %d images per call", kMaxTileColumns);
    P.bf16 = bf16;
    mfma_shape(L, L->n_panels, batch, dl.cus, bf16, P.nq, P.Bp, P.splits);
    P.lds = mfma_lds_bytes(L, bf16);
    if (P.lds > dl.max_lds) return fail(CL_EUNSUPPORTED, "the MFMA path needs %zu bytes of LDS", P.lds);
    P.xt_bytes = xt_bytes_for(L, P.Bp, bf16);
    P.part_bytes = (size_t)L->n_panels * P.splits * P.Bp * L->desc.block_h * sizeof(float);
    return CL_OK;
}

template <int NQ>
int32_t launch_mfma_as(const LayerDev &D, int panels, int splits, int np, int panels_per_x, size_t x_stride, size_t lds,
                       const float *xt, float *part, const DirectOut &out, hipStream_t st)
{
    static LdsLimit seen;
    if (int32_t rc = ensure_lds((const void *)fc_mfma_kernel<NQ>, lds, seen)) return rc;
    dim3 grid;
    GRID_TRY(grid, (int64_t)panels * splits * (np / MfmaShape<NQ>::kImages));
    hipLaunchKernelGGL(fc_mfma_kernel<NQ>, grid, dim3(MfmaShape<NQ>::kThreads), lds, st, D, xt, part, splits, np, panels_per_x, x_stride, out);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

template <int NQ>
int32_t launch_bf16_as(const LayerDev &D, int panels, int splits, int np, int panels_per_x, size_t x_stride, size_t lds,
                       const uint16_t *xb, size_t plane_elems, float *part, hipStream_t st)
{
    static LdsLimit seen;
    if (int32_t rc = ensure_lds((const void *)fc_mfma_bf16_kernel<NQ>, lds, seen)) return rc;
    dim3 grid;
    GRID_TRY(grid, (int64_t)panels * splits * (np / Bf16Shape<NQ>::kImages));
    hipLaunchKernelGGL(fc_mfma_bf16_kernel<NQ>, grid, dim3(Bf16Shape<NQ>::kThreads), lds, st, D, xb, part, splits, np, plane_elems, panels_per_x, x_stride);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

// panels block rows in one launch; each run of panels_per_x of them multiplies an
// activation matrix of its own, x_bytes after the one before
int32_t launch_mfma(const cl_layer *L, const LayerDev &D, bool bf16, int nq, int panels, int splits, int np, int panels_per_x,
                    size_t x_bytes, size_t lds, const void *xt, float *part, hipStream_t st,
                    const DirectOut &out = DirectOut{nullptr, nullptr, 0, 1, 0})
{
    const size_t x_stride = x_bytes / (bf16 ? sizeof(uint16_t) : sizeof(float));
    if (bf16) {
        const size_t pe = xb_plane_elems(L, np);
        switch (nq) {
        case 1: return launch_bf16_as<1>(D, panels, splits, np, panels_per_x, x_stride, lds, (const uint16_t *)xt, pe, part, st);
        case 2: return launch_bf16_as<2>(D, panels, splits, np, panels_per_x, x_stride, lds, (const uint16_t *)xt, pe, part, st);
        case 4: return launch_bf16_as<4>(D, panels, splits, np, panels_per_x, x_stride, lds, (const uint16_t *)xt, pe, part, st);
        case 8: return launch_bf16_as<8>(D, panels, splits, np, panels_per_x, x_stride, lds, (const uint16_t *)xt, pe, part, st);
        }
    } else {
        switch (nq) {
        case 1: return launch_mfma_as<1>(D, panels, splits, np, panels_per_x, x_stride, lds, (const float *)xt, part, out, st);
        case 2: return launch_mfma_as<2>(D, panels, splits, np, panels_per_x, x_stride, lds, (const float *)xt, part, out, st);
        case 4: return launch_mfma_as<4>(D, panels, splits, np, panels_per_x, x_stride, lds, (const float *)xt, part, out, st);
        case 8: return launch_mfma_as<8>(D, panels, splits, np, panels_per_x, x_stride, lds, (const float *)xt, part, out, st);
        }
    }
    return fail(CL_EINVAL, "internal: no dense-tile kernel for %d accumulators", nq);
}

// Launch shape of the wide sparse path (large batches on the vector ALUs).
struct WidePlan {
    int ipl = 4;             // images per lane: the image tile is 64 * ipl images
    int Bp = 0;              // batch rounded up to whole image tiles
    int splits = 1;          // workgroups sharing the blocks of one block row
    int64_t cost = 0;        // modelled cycles of the launches (same units as mfma_shape's)
    size_t lds = 0;
    size_t tile_bytes = 0;   // the partial tiles; behind them in the workspace's partial-tile part:
    size_t ent_bytes = 0;    //   the entry list
    size_t xt_bytes = 0, part_bytes = 0;
};

int32_t plan_wide(const cl_layer *L, int batch, const DeviceLimits &dl, WidePlan &P)
{
    if (!mfma_capable(L)) return fail(CL_EUNSUPPORTED, "the wide sparse path needs blocks of at most %d x %d", kTile, kTile);
    if (batch > kMaxTileColumns) return fail(CL_EUNSUPPORTED, "the wide sparse path takes at most %d images per call", kMaxTileColumns);
    P.ipl = batch > 128 ? 4 : batch > 64 ? 2 : 1;
    const int tile = 64 * P.ipl;
    P.Bp = (batch + tile - 1) / tile * tile;
    // two slabs of 64 columns x tile images, and the codebook
    P.lds = 2 * (size_t)kHalf * tile * sizeof(float) + ((size_t)4 << L->desc.weight_bits);
    if (P.lds > dl.max_lds) return fail(CL_EUNSUPPORTED, "the wide sparse path needs %zu bytes of LDS, %zu there", P.lds, dl.max_lds);
    // Split of the block rows, from a small model of the launches, in cycles per workgroup:
    // a start; per block two phases (one for blocks of at most 64 columns) of 2 k cycles and
    // a part per surviving weight - 9, 6.5 and 5.5 cycles at 4, 2 and 1 images per lane (at 4
    // the LDS port's 8 cycles per KB binds, below it the vector ALUs: 5 and 4 instructions
    // per weight over four SIMDs); the partial tiles, written and read again, as on the
    // dense-tile path; workgroups run in rounds of one per CU; and once per call the
    // decoding launch, 13 k and 6 per thousand entries.  Fitted to the AlexNet-shaped
    // fc6 / fc7 / fc8 at 256 images (multiply 68.7 / 35.1 / 24.8 us, decode 16.2 / 8.5 / 8.0 us; the decoding launch has become
    // shorter since.  Over the calls of plan_rows 0.41 us to a thousand cycles, rms 10 %).
    const int64_t tiles = (int64_t)L->n_panels * (P.Bp / tile);
    const int cus = std::max(1, dl.cus);
    const int64_t nnz_block = L->n_blocks ? L->nnz / L->n_blocks : 0;
    const int64_t per_weight_x2 = P.ipl == 4 ? 18 : P.ipl == 2 ? 13 : 11;
    const int64_t per_block = (L->desc.block_w > kHalf ? 4000 : 2000) + nnz_block * per_weight_x2 / 2;
    const int64_t start = 12000, once = 13000 + L->entries * 6 / 1000;
    const int sp_max = (int)std::max<int64_t>(1, std::min<int64_t>(L->nbw, (3 * (int64_t)cus + tiles - 1) / tiles));
    int64_t best = -1;
    for (int sp = 1; sp <= sp_max; ++sp) {
        const int64_t rounds = (tiles * sp + cus - 1) / cus, blocks = (L->nbw + sp - 1) / sp;
        const int64_t t = once + rounds * (start + blocks * per_block) +
                          (int64_t)L->n_panels * sp * P.Bp * kTile * (int64_t)sizeof(float) * 3 / 4000;
        if (best < 0 || t < best) {
            best = t;
            P.splits = sp;
        }
    }
    P.cost = best;
    P.xt_bytes = xt_bytes_for(L, P.Bp, false);
    P.tile_bytes = (size_t)L->n_panels * P.splits * kTile * P.Bp * sizeof(float);
    P.ent_bytes = ((size_t)L->nnz * sizeof(WideEntry) + 255) / 256 * 256;
    P.part_bytes = P.tile_bytes + P.ent_bytes;
    return CL_OK;
}

template <int IPL>
int32_t launch_wide_mul(const LayerDev &D, int panels, const WidePlan &P, const float *xt, float *part, const WideEntry *ent,
                        hipStream_t st)
{
    static LdsLimit seen;
    if (int32_t rc = ensure_lds((const void *)wide_mul_kernel<IPL>, P.lds, seen)) return rc;
    dim3 grid;
    GRID_TRY(grid, (int64_t)panels * P.splits * (P.Bp / (64 * IPL)));
    hipLaunchKernelGGL(wide_mul_kernel<IPL>, grid, dim3(kWideThreads), P.lds, st, D, xt, ent, part, panels, P.splits, P.Bp);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

// CL_PATH_AUTO: the sparse path up to kAutoSparseBatch images (one batch tile of its small-batch
// kernel) and for blocks above 128 x 128; above, whichever of the sparse path's fc_rows_kernel,
// the dense-tile path and the wide sparse path their launch models price lower (same units, all
// fitted to measured launches).  fc_rows_kernel is taken up to kAutoLaunch cycles above the others: the launch it saves,
// which lays the activations out or decodes (2.5 us, 6 k cycles, in the fits of the three paths), and a part of what its price is
// too high by (plan_rows).  Over the 1400 calls measured there the choice is 2.1 % slower on average than the best of the three
// paths, more than 5 % in 139; with 6 k cycles 2.5 % and 180, and all 44 calls whose path differs are slower with 6 k, by 1 to 53 %.  (With the price
// at 7/8 and 6 k cycles 1.4 % and 75; but of 600 calls of stacks of such layers 26 become slower, by up to 7.5 %, and 36 faster, by up to 10 %:
// choose_stack_paths weighs all of a stack's layers that would be on fc_rows_kernel against none of them.)  AlexNet-shaped stack (fc6 / fc7 / fc8, us per layer call): small-batch kernel
// 24 / 16 / 14 at 8 images; at 16 images fc_rows_kernel 24 / 16 / 12, dense tiles 40 / 24 / 18; at 64 images 41 / 25 / 17 and
// 60 / 35 / 23; at 128 images 71 / 40 / 24, wide 73 / 47 / 41 (fc6 is on the latter); at 256 images 128 / 66 / 36, wide 91 / 55 / 47,
// dense tiles 163 / 88 / 40 (fc8 is on these) - the dense tile multiplies eleven times the necessary
// products at a 9 % density but four at 25 %.  A layer of fewer than kAutoRowsBlocks blocks takes
// 12 to 16 us on either, launches for the most part, and stays on dense tiles.  (Where the sparse path
// runs the small-batch kernel instead, rows_kernel_pays, that is the cheaper one: the price is an upper bound.)
constexpr int kAutoSparseBatch = 8;
constexpr int kAutoRowsBlocks = 48;
constexpr int64_t kAutoLaunch = 9000;

// How one layer runs for a batch: the path, and that path's launch shape.  Made once per call (what
// the choice of a path has worked out for it is kept).
struct FcPlan {
    int path = 0;
    bool have_wide = false, have_rows = false;      // left by the choice: wide, sparse.rows
    int no_rows = 0;                                // and the path it would be without fc_rows_kernel (0: it is not that kernel)
    int64_t mfma_cost = 0, rows_cost = 0;
    SparsePlan sparse;
    MfmaPlan mfma;
    WidePlan wide;
    size_t bytes() const { return path == CL_PATH_SPARSE ? sparse.part_bytes : path == CL_PATH_SPARSE_WIDE ? wide.xt_bytes + wide.part_bytes : mfma.xt_bytes + mfma.part_bytes; }
};

void choose_path(const cl_layer *L, int batch, int path, const DeviceLimits &dl, FcPlan &P)
{
    P.path = path;
    if (path != CL_PATH_AUTO) return;
    P.path = CL_PATH_SPARSE;
    if (batch <= kAutoSparseBatch || !mfma_capable(L)) return;
    P.path = CL_PATH_MFMA_F32;
    if (batch > kMaxTileColumns) return;                    // refused there with its message
    int nq, np, splits;
    int64_t best = 0;
    mfma_shape(L, L->n_panels, batch, dl.cus, false, nq, np, splits, false, false, &best);
    P.mfma_cost = best;
    P.have_wide = plan_wide(L, batch, dl, P.wide) == CL_OK;
    if (!P.have_wide) clear_error();
    else if (P.wide.cost < best) {
        best = P.wide.cost;
        P.path = CL_PATH_SPARSE_WIDE;
    }
    P.have_rows = L->n_blocks >= kAutoRowsBlocks && plan_rows(L, batch, dl, P.sparse.rows);
    P.rows_cost = P.sparse.rows.cost;
    if (P.have_rows && P.rows_cost < best + kAutoLaunch) {
        P.no_rows = P.path;
        P.path = CL_PATH_SPARSE;
    }
}

bool is_mfma(int path) { return path == CL_PATH_MFMA_F32 || path == CL_PATH_MFMA_BF16; }

// the paths that read the activations transposed and laid out block by block
bool reads_xt(int path) { return is_mfma(path) || path == CL_PATH_SPARSE_WIDE; }

int32_t plan_fc(const cl_layer *L, int batch, int path, const DeviceLimits &dl, FcPlan &P)
{
    if (batch < 1) return fail(CL_EINVAL, "batch must be positive");
    if (path < CL_PATH_AUTO || path > CL_PATH_SPARSE_WIDE) return fail(CL_EINVAL, "unknown path %d", path);
    choose_path(L, batch, path, dl, P);
    if (P.path == CL_PATH_SPARSE_WIDE) return P.have_wide ? (int32_t)CL_OK : plan_wide(L, batch, dl, P.wide);
    if (is_mfma(P.path)) return plan_mfma(L, batch, P.path == CL_PATH_MFMA_BF16, dl, P.mfma);
    const RowsPlan rows = P.sparse.rows;
    P.sparse = SparsePlan{};
    return plan_sparse(L, batch, dl, P.sparse, false, P.have_rows ? &rows : nullptr);
}

}  // namespace

extern "C" int32_t cl_fc_workspace_bytes(const cl_layer *L, int32_t batch, int32_t path, size_t *out)
{
    if (!L || !out) return fail(CL_EINVAL, "null argument");
    if (batch < 1) return fail(CL_EINVAL, "batch must be positive");
    if (path < CL_PATH_AUTO || path > CL_PATH_SPARSE_WIDE) return fail(CL_EINVAL, "unknown path %d", path);
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    FcPlan P;
    if (int32_t rc = plan_fc(L, batch, path, dl, P)) return rc;
    *out = P.bytes();
    return CL_OK;
}

extern "C" int32_t cl_fc_resolved_path(const cl_layer *L, int32_t batch, int32_t path, int32_t *out)
{
    if (!L || !out) return fail(CL_EINVAL, "null argument");
    if (batch < 1) return fail(CL_EINVAL, "batch must be positive");
    if (path < CL_PATH_AUTO || path > CL_PATH_SPARSE_WIDE) return fail(CL_EINVAL, "unknown path %d", path);
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    FcPlan P;
    choose_path(L, batch, path, dl, P);
    *out = P.path;
    return CL_OK;
}

template <int IPL, int G>
static int32_t launch_rows(const LayerDev &D, int panels, const RowsPlan &P, const float *d_X, float *part, int batch, hipStream_t st)
{
    const int Bp = P.padded(batch);
    static LdsLimit seen;
    if (int32_t rc = ensure_lds((const void *)fc_rows_kernel<IPL, G>, P.lds, seen)) return rc;
    dim3 grid;
    GRID_TRY(grid, (int64_t)panels * P.splits * (Bp / (16 * IPL)));
    hipLaunchKernelGGL((fc_rows_kernel<IPL, G>), grid, dim3(kRowsThreads), P.lds, st, D, d_X, part, batch, panels, P.splits, Bp, P.list_cap);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

// One layer through fc_rows_kernel with launch shape P, and its finishing kernel; run after run
// through the same partial tiles.
static int32_t forward_rows(const cl_layer *L, const LayerDev &D, const RowsPlan &P, const float *d_X, const float *d_bias, float *d_Y,
                            int batch, int relu, float *part, hipStream_t st)
{
    for (int b0 = 0; b0 < batch; b0 += P.run) {
        const int nb = std::min(P.run, batch - b0), Bp = P.padded(nb);
        const float *x = d_X + (size_t)b0 * L->desc.K;
        if (b0 == 0) timing_begin(st);      // benchmarks time the first main-kernel launch of a call
        int32_t rc = CL_EINVAL;
        switch (P.ipl * 8 + P.group) {
        case 1 * 8 + 1: rc = launch_rows<1, 1>(D, L->n_panels, P, x, part, nb, st); break;
        case 1 * 8 + 2: rc = launch_rows<1, 2>(D, L->n_panels, P, x, part, nb, st); break;
        case 1 * 8 + 4: rc = launch_rows<1, 4>(D, L->n_panels, P, x, part, nb, st); break;
        case 2 * 8 + 1: rc = launch_rows<2, 1>(D, L->n_panels, P, x, part, nb, st); break;
        case 2 * 8 + 2: rc = launch_rows<2, 2>(D, L->n_panels, P, x, part, nb, st); break;
        case 2 * 8 + 3: rc = launch_rows<2, 3>(D, L->n_panels, P, x, part, nb, st); break;
        case 4 * 8 + 1: rc = launch_rows<4, 1>(D, L->n_panels, P, x, part, nb, st); break;
        }
        if (rc) return rc;
        if (b0 == 0) timing_end(st, 1);
        dim3 rgrid;
        const int quads = rows_reduce_quads(Bp), rows = kRowsRedPieces / quads;
        GRID_TRY(rgrid, (int64_t)((L->desc.M + rows - 1) / rows) * (Bp / (4 * quads)));
        hipLaunchKernelGGL(rows_reduce_kernel, rgrid, dim3(kRowsRedParts * kRowsRedPieces), 0, st, D, part, d_bias, d_Y + (size_t)b0 * L->desc.M, nb, Bp, P.splits, relu);
        HIP_TRY(hipGetLastError());
    }
    return CL_OK;
}

// One layer on the sparse path with launch shape P.  With `prev` the input is not d_X but the partial
// tiles of the layer before (see PrevSlots); with finish == false the layer's own
// finishing kernel is left to the layer after it in the same way.  Both only where
// sparse_can_fold allows.  in_stack: other layers' launches come before or behind.
static int32_t forward_sparse(const cl_layer *L, const LayerDev &D, const SparsePlan &P, const float *d_X,
                              const float *d_bias, float *d_Y, int batch, int relu, float *part, hipStream_t st,
                              bool in_stack = false, const PrevSlots *prev = nullptr, bool finish = true)
{
    if (P.rows.ipl) return forward_rows(L, D, P.rows, d_X, d_bias, d_Y, batch, relu, part, st);
    const PrevSlots from = prev ? *prev : PrevSlots{};
    if ((prev || !finish) && !sparse_can_fold(L, P, batch)) return fail(CL_EINVAL, "internal: layer cannot take or leave partial tiles");
    const int M = L->desc.M, K = L->desc.K;
    dim3 grid;
    if (L->n_chunks > 0) GRID_TRY(grid, (int64_t)L->n_panels * P.wg_per_panel);
    const auto alone = [&]() {
        hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
        if (in_stack || batch > P.bt_max) return false;
        if (hipStreamIsCapturing(st, &capture) == hipSuccess) return capture == hipStreamCaptureStatusNone;
        (void)hipGetLastError();
        return false;
    };
    for (int b0 = 0; b0 < batch;) {
        // the smallest batch tile that holds the images left (its other images are zeros):
        // one launch for 3 images, not two
        const int nb = std::min(P.bt_max, batch - b0);
        int bt = P.bt_max;
        while (bt / 2 >= nb) bt >>= 1;
        const float *x = d_X + (size_t)b0 * K;
        float *y = d_Y + (size_t)b0 * M;
        const size_t whole = finish && !prev && L->n_chunks > 0 ? P.whole_lds(L, bt, alone) : 0;
        if (whole) {
            const WholeOut out{d_bias, y, relu};
            dim3 rows;
            GRID_TRY(rows, L->n_panels);
            if (b0 == 0) timing_begin(st);
            switch (bt) {
            case 4: hipLaunchKernelGGL(fc_sparse_whole_kernel<4>, rows, dim3(kWholeWaves * 64), whole, st, D, x, out, nb); break;
            case 2: hipLaunchKernelGGL(fc_sparse_whole_kernel<2>, rows, dim3(kWholeWaves * 64), whole, st, D, x, out, nb); break;
            default: hipLaunchKernelGGL(fc_sparse_whole_kernel<1>, rows, dim3(kWholeWaves * 64), whole, st, D, x, out, nb); break;
            }
            HIP_TRY(hipGetLastError());
            if (b0 == 0) timing_end(st, 1);
        } else if (L->n_chunks > 0) {
            const size_t lds = P.lds_for(L, bt);
            const int xcap = P.xcap_for(bt);
            if (b0 == 0) timing_begin(st);      // benchmarks time the first main-kernel launch of a call
#define CL_LAUNCH_SPARSE(BTV, FOLDV)                                                                               \
    do {                                                                                                           \
        if (lds > 64 * 1024)                                                                                       \
            HIP_TRY(hipFuncSetAttribute((const void *)fc_sparse_kernel<BTV, FOLDV>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)); \
        hipLaunchKernelGGL((fc_sparse_kernel<BTV, FOLDV>), grid, dim3(kThreads), lds, st, D, x, part, divisor((uint32_t)P.wg_per_panel), xcap, from, nb); \
    } while (0)
            switch (bt) {
            case 16: CL_LAUNCH_SPARSE(16, false); break;
            case 8: CL_LAUNCH_SPARSE(8, false); break;
            case 4: CL_LAUNCH_SPARSE(4, false); break;
            case 2: CL_LAUNCH_SPARSE(2, false); break;
            default:
                if (prev) CL_LAUNCH_SPARSE(1, true);
                else CL_LAUNCH_SPARSE(1, false);
                break;
            }
#undef CL_LAUNCH_SPARSE
            HIP_TRY(hipGetLastError());
            if (b0 == 0) timing_end(st, 1);
        }
        if (finish && !whole) {
            dim3 rgrid;
            GRID_TRY(rgrid, (int64_t)L->n_panels * nb);
            hipLaunchKernelGGL(fc_reduce_kernel, rgrid, dim3(kRedThreads), 0, st,
                               D, part, d_bias, y, nb, bt, P.wg_per_panel, relu);
            HIP_TRY(hipGetLastError());
        }
        b0 += nb;
    }
    return CL_OK;
}

// One layer on a dense-tile path with launch shape P.  The input is d_X (batch x K, laid
// out for the kernel into xt first) or, when d_X is null, already sits in xt.  The
// output goes to d_Y as batch x M, or, with next_bp > 0, as the transposed activations
// of a following 128-column-block layer whose image axis is padded to next_bp
// (Y[row][next_bp], padded images zero; on the bf16 path its two planes).
static int32_t run_mfma_layer(const cl_layer *L, const LayerDev &D, const MfmaPlan &P, const float *d_X, void *xt, float *part,
                              const float *d_bias, float *d_Y, int next_bp, int batch, int relu, hipStream_t st)
{
    const int K = L->desc.K;
    if (d_X) {
        if (P.bf16) {
            hipLaunchKernelGGL(split_pad_kernel, dim3((unsigned)(L->nbw * 8), (unsigned)((P.Bp + 63) / 64)), dim3(256), 0, st,
                               d_X, (uint16_t *)xt, batch, K, P.Bp, L->desc.block_w, xb_plane_elems(L, P.Bp));
        } else {
            const int rows = L->nbw * kTile;
            hipLaunchKernelGGL(transpose_pad_kernel, dim3((unsigned)(rows / 32), (unsigned)(P.Bp / 32)), dim3(256), 0, st,
                               d_X, (float *)xt, batch, K, P.Bp, L->desc.block_w, rows);
        }
        HIP_TRY(hipGetLastError());
    }
    timing_begin(st);
    if (int32_t rc = launch_mfma(L, D, P.bf16, P.nq, L->n_panels, P.splits, P.Bp, L->n_panels, 0, P.lds, xt, part, st)) return rc;
    timing_end(st, 1);
    if (P.bf16 && next_bp > 0) {
        dim3 grid;
        GRID_TRY(grid, ((int64_t)(L->desc.M / 4) * next_bp + 255) / 256);
        hipLaunchKernelGGL(bf16_reduce_kernel, grid, dim3(256), 0, st, D, part, d_bias, (uint16_t *)d_Y, batch, P.Bp, P.splits, relu, next_bp,
                           ((size_t)(L->desc.M / kTile) * 8 + kXbTailGroups) * next_bp * 16);       // (xb_plane_elems of the next layer)
        HIP_TRY(hipGetLastError());
        return CL_OK;
    }
    const int cols = std::max(batch, next_bp);
    // towards a following layer the output runs along the images: full 32-column tiles
    // (128-byte runs), and the rows of a block row shared out to keep the launch wide
    int ct = reduce_col_tile(L->n_panels, cols), rt = L->desc.block_h;
    if (next_bp > 0) {
        ct = kColTile;
        rt = kTile;
        while (rt > 32 && (int64_t)L->n_panels * ((cols + ct - 1) / ct) * ((L->desc.block_h + rt - 1) / rt) < 1024) rt >>= 1;
    }
    const int nrt = (L->desc.block_h + rt - 1) / rt;
    dim3 rgrid;
    GRID_TRY(rgrid, (int64_t)L->n_panels * ((cols + ct - 1) / ct) * nrt);
    hipLaunchKernelGGL(mfma_reduce_kernel, rgrid, dim3(256), 0, st,
                       D, part, d_bias, d_Y, batch, P.Bp, P.splits, relu, next_bp, ct, next_bp, rt);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

// The decoding launch of the wide path for up to kExpandJobs layers at once, each
// into its own list.  Layers without chunks are skipped (their lists are empty).
// (xt_of: the layer whose activations d_X, batch x K, the launch lays out as well, into xt
// with the image axis padded to bp - or null)
static int32_t launch_wide_expand(const cl_layer *const *layers, WideEntry *const *ents, int n, int ipl, hipStream_t st,
                                  const cl_layer *xt_of = nullptr, const float *d_X = nullptr, float *xt = nullptr, int batch = 0,
                                  int bp = 0)
{
    ExpandJobs jobs{};
    jobs.ipl = (uint32_t)ipl;
    size_t lds = xt_of ? kExpandTurnBytes : 0;
    int64_t wgs = 0, t_wgs = 0;
    int used = 0;
    if (xt_of) {
        jobs.X = d_X;
        jobs.XT = xt;
        jobs.B = batch;
        jobs.K = xt_of->desc.K;
        jobs.Bp = bp;
        jobs.bw = xt_of->desc.block_w;
        jobs.rows = xt_of->nbw * kTile;
        t_wgs = ((int64_t)(jobs.rows / 32) * (bp / 32) + 1) / 2;
    }
    for (int i = 0; i < n; ++i) {
        const cl_layer *L = layers[i];
        if (L->n_chunks == 0) continue;
        jobs.L[used] = make_dev(L);
        jobs.ent[used] = ents[i];
        jobs.wg0[used] = (uint32_t)wgs;
        wgs += (L->n_chunks + kWaves - 1) / kWaves;
        lds = std::max(lds, table_image_bytes(L->val_lut_bits, L->idx_lut_bits, 1 << L->desc.weight_bits) + kWaves * kExpandList * sizeof(uint32_t));
        ++used;
    }
    if (!used && !t_wgs) return CL_OK;
    jobs.t_wg0 = (uint32_t)wgs;
    for (int i = used; i <= kExpandJobs; ++i) jobs.wg0[i] = i == used ? (uint32_t)wgs : UINT32_MAX;
    if (!used) {
        // nothing to decode: the launch only lays the activations out (the job table names the
        // first layer, whose range of workgroups is empty)
        jobs.L[0] = make_dev(xt_of);
        jobs.wg0[0] = (uint32_t)wgs;
    }
    for (int i = std::max(used, 1); i < kExpandJobs; ++i) jobs.L[i] = jobs.L[0];
    static LdsLimit seen;
    if (int32_t rc = ensure_lds((const void *)wide_expand_kernel, lds, seen)) return rc;
    dim3 egrid;
    GRID_TRY(egrid, wgs + t_wgs);
    hipLaunchKernelGGL(wide_expand_kernel, egrid, dim3(kThreads), lds, st, jobs);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

// One layer on the wide sparse path with launch shape P; arguments as run_mfma_layer.  The
// entry list is `ent`; with expanded it has been written already (by a launch_wide_expand
// that took several layers of a stack together).
static int32_t run_wide_layer(const cl_layer *L, const LayerDev &D, const WidePlan &P, const float *d_X, float *xt, float *part,
                              WideEntry *ent, bool expanded, const float *d_bias, float *d_Y, int next_bp, int batch, int relu,
                              hipStream_t st)
{
    int32_t rc = CL_EINVAL;
    if (!expanded) {
        // one launch decodes the layer and lays its activations out
        if ((rc = launch_wide_expand(&L, &ent, 1, P.ipl, st, d_X ? L : nullptr, d_X, xt, batch, P.Bp))) return rc;
    } else if (d_X) {
        const int rows = L->nbw * kTile;
        hipLaunchKernelGGL(transpose_pad_kernel, dim3((unsigned)(rows / 32), (unsigned)(P.Bp / 32)), dim3(256), 0, st,
                           d_X, xt, batch, L->desc.K, P.Bp, L->desc.block_w, rows);
        HIP_TRY(hipGetLastError());
    }
    timing_begin(st);
    switch (P.ipl) {
    case 1: rc = launch_wide_mul<1>(D, L->n_panels, P, xt, part, ent, st); break;
    case 2: rc = launch_wide_mul<2>(D, L->n_panels, P, xt, part, ent, st); break;
    case 4: rc = launch_wide_mul<4>(D, L->n_panels, P, xt, part, ent, st); break;
    }
    if (rc) return rc;
    timing_end(st, 1);
    const int ncol = std::max(P.Bp, next_bp);
    dim3 rgrid;
    GRID_TRY(rgrid, (int64_t)L->n_panels * (kTile / kWideRedRows) * ((ncol + kWideRedImages - 1) / kWideRedImages));
    hipLaunchKernelGGL(wide_reduce_kernel, rgrid, dim3(256), 0, st, D, part, d_bias, d_Y, batch, P.Bp, P.splits, relu, next_bp);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

// The checks of a single-layer call (before anything is planned), then its launches with plan P.
static int32_t check_fc_call(const cl_layer *L, const float *d_X, const float *d_Y, int32_t batch)
{
    if (int32_t rc = require_device(L)) return rc;
    if (!d_X || !d_Y) return fail(CL_EINVAL, "null activation pointer");
    if (batch < 1) return fail(CL_EINVAL, "batch must be positive");
    return CL_OK;
}

static int32_t forward_planned(const cl_layer *L, const FcPlan &P, const float *d_X, const float *d_bias, float *d_Y, int32_t batch,
                               int32_t relu, void *d_workspace, size_t workspace_bytes, hipStream_t st)
{
    const size_t need = P.bytes();
    if (workspace_bytes < need || (need && !d_workspace)) return fail(CL_EINVAL, "workspace too small: %zu < %zu", workspace_bytes, need);
    if ((uintptr_t)d_workspace % 256) return fail(CL_EINVAL, "workspace must be 256-byte aligned");
    const LayerDev D = make_dev(L);
    char *ws = (char *)d_workspace;
    int32_t rc;
    if (P.path == CL_PATH_SPARSE_WIDE)
        rc = run_wide_layer(L, D, P.wide, d_X, (float *)ws, (float *)(ws + P.wide.xt_bytes), (WideEntry *)(ws + P.wide.xt_bytes + P.wide.tile_bytes), false,
                            d_bias, d_Y, 0, batch, relu, st);
    else if (is_mfma(P.path))
        rc = run_mfma_layer(L, D, P.mfma, d_X, ws, (float *)(ws + P.mfma.xt_bytes), d_bias, d_Y, 0, batch, relu, st);
    else
        rc = forward_sparse(L, D, P.sparse, d_X, d_bias, d_Y, batch, relu, (float *)ws, st);
    if (rc == CL_OK) clear_error();
    return rc;
}

extern "C" int32_t cl_compressed_fc_forward(const cl_layer *L, const float *d_X, const float *d_bias,
                                            float *d_Y, int32_t batch, int32_t relu, int32_t path,
                                            void *d_workspace, size_t workspace_bytes, void *stream)
{
    if (int32_t rc = check_fc_call(L, d_X, d_Y, batch)) return rc;
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    FcPlan P;
    if (int32_t rc = plan_fc(L, batch, path, dl, P)) return rc;
    return forward_planned(L, P, d_X, d_bias, d_Y, batch, relu, d_workspace, workspace_bytes, (hipStream_t)stream);
}

extern "C" int32_t cl_compressed_fc_forward_static(const cl_layer *L, const float *d_X, const float *d_bias,
                                                   float *d_Y, int32_t batch, int32_t relu, int32_t path, void *stream)
{
    if (int32_t rc = check_fc_call(L, d_X, d_Y, batch)) return rc;
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    FcPlan P;
    if (int32_t rc = plan_fc(L, batch, path, dl, P)) return rc;
    if (P.bytes() > (size_t)CL_STATIC_SCRATCH_BYTES)
        return fail(CL_EUNSUPPORTED, "this call needs %zu bytes of scratch, the static scratch area holds %zu: use cl_compressed_fc_forward with a workspace",
                    P.bytes(), (size_t)CL_STATIC_SCRATCH_BYTES);
    void *scratch = nullptr;
    if (int32_t rc = static_scratch(&scratch)) return rc;
    return forward_planned(L, P, d_X, d_bias, d_Y, batch, relu, scratch, (size_t)CL_STATIC_SCRATCH_BYTES, (hipStream_t)stream);
}

// ------------------------------------------------------------------------- //
// a stack of fully connected layers (Eq. 1 layer after layer)
// ------------------------------------------------------------------------- //
namespace {

struct StackPlan {
    std::vector<FcPlan> fc;           // per layer: the path it runs on, and its launch shape
    std::vector<char> xt_in;          // layer reads its transposed activations straight from the layer before
    std::vector<char> fold_in;        // layer adds up the partial tiles of the layer before itself (both on the sparse path)
    std::vector<size_t> ent_off;      // per layer on the wide path: its entry list in the area behind the rotating buffers
    size_t xt_bytes = 0, part_bytes = 0, act_bytes = 0, ent_bytes = 0;
    int regions = 1;                  // copies of each buffer, used in rotation
    size_t total() const { return (size_t)regions * (xt_bytes + part_bytes + act_bytes) + ent_bytes; }
};

size_t round256(size_t n) { return (n + 255) / 256 * 256; }

constexpr int kStackRegions = 4;

// Whether the finishing kernel of the layer before can write this layer's transposed
// activations itself: when their row order is the plain one (128-column blocks, no ragged
// last block): 2-3 % of a step on the AlexNet-shaped stack.
bool plain_rows(const cl_layer *L) { return L->desc.block_w == kTile && L->desc.K % kTile == 0; }

// CL_PATH_AUTO for the layers of a stack.  What fc_rows_kernel saves a single layer - the launch that
// lays the activations out, or decodes - a layer between two on the other paths does not pay: its
// neighbour hands the activations over, and one launch decodes all layers on the wide path.  So where
// some layers run on fc_rows_kernel and some do not, the modelled cycles of the whole stack decide
// whether the former do without it (us a step, AlexNet- and VGG-shaped stack: at 128 images, fc6 wide either way,
// 144 and 161 with fc_rows_kernel for fc7 and fc8, 136 and 156 without; at 64, all three layers on it, 81 and 106,
// 115 and 136 without).
constexpr int64_t kWideShared = 13000;          // the decoding launch's fixed part (plan_wide)

void choose_stack_paths(const cl_layer *const *layers, int n, int batch, const DeviceLimits &dl, std::vector<FcPlan> &fc)
{
    bool some = false, others = false;
    for (const FcPlan &P : fc) (P.no_rows ? some : others) = true;
    if (!some || !others) return;
    auto cost = [&](bool rows) {
        int64_t t = 0;
        bool wide = false, before = false;      // a wide layer yet; the layer before hands activations over
        for (int i = 0; i < n; ++i) {
            const FcPlan &P = fc[i];
            const int path = rows || !P.no_rows ? P.path : P.no_rows;
            const bool handed = before && plain_rows(layers[i]);
            if (path == CL_PATH_SPARSE) t += P.no_rows ? P.rows_cost : 0;
            else if (path == CL_PATH_SPARSE_WIDE) t += P.wide.cost - (wide ? kWideShared : 0) + (i > 0 && !handed ? kAutoLaunch : 0);
            else t += P.mfma_cost + (handed ? 0 : kAutoLaunch);
            wide = wide || path == CL_PATH_SPARSE_WIDE;
            before = reads_xt(path);
        }
        return t;
    };
    if (cost(true) <= cost(false)) return;
    for (int i = 0; i < n; ++i)
        if (const int path = fc[i].no_rows) {
            FcPlan without;
            if (plan_fc(layers[i], batch, path, dl, without) == CL_OK) fc[i] = without;
            else clear_error();                 // (a layer that path does not fit: it stays)
        }
}

int32_t plan_stack(const cl_layer *const *layers, int n, int batch, int path, const DeviceLimits &dl, StackPlan &P)
{
    if (!layers || n < 1) return fail(CL_EINVAL, "a stack needs at least one layer");
    if (batch < 1) return fail(CL_EINVAL, "batch must be positive");
    if (path < CL_PATH_AUTO || path > CL_PATH_SPARSE_WIDE) return fail(CL_EINVAL, "unknown path %d", path);
    P.fc.assign(n, FcPlan{});
    P.xt_in.assign(n, 0);
    P.fold_in.assign(n, 0);
    P.ent_off.assign(n, 0);
    for (int i = 0; i < n; ++i) {
        const cl_layer *L = layers[i];
        if (!L) return fail(CL_EINVAL, "layer %d is null", i);
        if (i > 0 && L->desc.K != layers[i - 1]->desc.M)
            return fail(CL_EINVAL, "layer %d takes %d inputs, layer %d gives %d outputs", i, L->desc.K, i - 1, layers[i - 1]->desc.M);
        if (int32_t rc = plan_fc(L, batch, path, dl, P.fc[i])) return rc;
    }
    if (path == CL_PATH_AUTO) choose_stack_paths(layers, n, batch, dl, P.fc);
    for (int i = 0; i < n; ++i) {
        const cl_layer *L = layers[i];
        const int mine = P.fc[i].path, before = i > 0 ? P.fc[i - 1].path : 0;
        if (mine == CL_PATH_SPARSE_WIDE) {
            P.xt_bytes = std::max(P.xt_bytes, P.fc[i].wide.xt_bytes);
            P.part_bytes = std::max(P.part_bytes, round256(P.fc[i].wide.tile_bytes));
            P.ent_off[i] = P.ent_bytes;
            P.ent_bytes += round256(P.fc[i].wide.ent_bytes);
            P.xt_in[i] = i > 0 && reads_xt(before) && plain_rows(L);
        } else if (is_mfma(mine)) {
            P.xt_bytes = std::max(P.xt_bytes, P.fc[i].mfma.xt_bytes);
            P.part_bytes = std::max(P.part_bytes, round256(P.fc[i].mfma.part_bytes));
            P.xt_in[i] = i > 0 && plain_rows(L) && (mine == CL_PATH_MFMA_F32 ? reads_xt(before) : before == CL_PATH_MFMA_BF16 && layers[i - 1]->desc.block_h % 4 == 0);
        } else {
            P.part_bytes = std::max(P.part_bytes, round256(P.fc[i].sparse.part_bytes));
            // (measured on the AlexNet-shaped stack: 39.8 -> 37.1 us at one image, no gain at
            // two, a loss at four - every workgroup of a block column adds the same tiles up)
            P.fold_in[i] = batch == 1 && i > 0 && before == CL_PATH_SPARSE && sparse_can_fold(layers[i - 1], P.fc[i - 1].sparse, batch) &&
                           sparse_can_fold(L, P.fc[i].sparse, batch);
        }
        if (i + 1 < n) P.act_bytes = std::max(P.act_bytes, round256((size_t)batch * L->desc.M * sizeof(float)));
    }
    P.regions = std::min(n, kStackRegions);
    return CL_OK;
}

}  // namespace

extern "C" int32_t cl_fc_stack_workspace_bytes(const cl_layer *const *layers, int32_t n_layers, int32_t batch, int32_t path,
                                               size_t *out)
try {
    if (!out) return fail(CL_EINVAL, "null argument");
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    StackPlan P;
    if (int32_t rc = plan_stack(layers, n_layers, batch, path, dl, P)) return rc;
    *out = P.total();
    return CL_OK;
} catch (...) {
    return fail_with_exception();
}

extern "C" int32_t cl_compressed_fc_stack_forward(const cl_layer *const *layers, int32_t n_layers, const float *d_X,
                                                  const float *const *d_bias_or_null, float *d_Y, int32_t batch,
                                                  int32_t relu_hidden, int32_t relu_last, int32_t path, void *d_workspace,
                                                  size_t workspace_bytes, void *stream)
try {
    if (!d_X || !d_Y) return fail(CL_EINVAL, "null activation pointer");
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    StackPlan P;
    if (int32_t rc = plan_stack(layers, n_layers, batch, path, dl, P)) return rc;
    for (int i = 0; i < n_layers; ++i)
        if (int32_t rc = require_device(layers[i])) return rc;
    if (workspace_bytes < P.total() || (P.total() && !d_workspace))
        return fail(CL_EINVAL, "workspace too small: %zu < %zu", workspace_bytes, P.total());
    if ((uintptr_t)d_workspace % 256) return fail(CL_EINVAL, "workspace must be 256-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)d_workspace;
    // Up to four of everything, used in rotation.  Two would do for the data's lifetime;
    // more are a matter of speed: a kernel that writes where a kernel shortly before has
    // read (the partial tiles above all) runs slower, the lines being still held by the
    // other dies' caches - 3 % of a step at batch 256 with one buffer of partial tiles,
    // 5 % at batch 64 with two.
    const int R = P.regions;
    auto region = [&](size_t base, size_t bytes, int i) { return ws + base + (size_t)(i % R) * bytes; };
    const size_t xt0 = 0, part0 = (size_t)R * P.xt_bytes, act0 = part0 + (size_t)R * P.part_bytes;
    // The layers on the wide path are decoded up front, kExpandJobs to a launch: the
    // lists depend on the weights only, and one launch for two layers is shorter than two
    // (the fixed part of such a launch - start, tables, the dependent loads - is a third of fc7's).
    const size_t ent0 = act0 + (size_t)R * P.act_bytes;
    auto ent_of = [&](int i) { return (WideEntry *)(ws + ent0 + P.ent_off[i]); };
    // (the first of these launches also lays out the input of the stack when its first layer is
    // one of them)
    bool x_laid_out = false;
    {
        const cl_layer *todo[kExpandJobs];
        WideEntry *ents[kExpandJobs];
        int n = 0, ipl_of_stack = 4;                 // (the images per lane follow from the batch: the same for every layer)
        for (int i = 0; i <= n_layers; ++i) {
            const bool mine = i < n_layers && P.fc[i].path == CL_PATH_SPARSE_WIDE;
            if (mine) {
                todo[n] = layers[i];
                ents[n] = ent_of(i);
                ipl_of_stack = P.fc[i].wide.ipl;
                ++n;
            }
            if (n == kExpandJobs || (i == n_layers && n > 0)) {
                const bool with_x = !x_laid_out && P.fc[0].path == CL_PATH_SPARSE_WIDE;
                if (int32_t rc = launch_wide_expand(todo, ents, n, ipl_of_stack, st, with_x ? layers[0] : nullptr, d_X,
                                                    (float *)region(xt0, P.xt_bytes, 0), batch, P.fc[0].wide.Bp))
                    return rc;
                x_laid_out = x_laid_out || with_x;
                n = 0;
            }
        }
    }
    const float *in = x_laid_out ? nullptr : d_X;    // the layer's input as batch x K, or null when it sits in its xt region
    for (int i = 0; i < n_layers; ++i) {
        const cl_layer *L = layers[i];
        const LayerDev D = make_dev(L);
        const bool last = i + 1 == n_layers;
        const float *bias = d_bias_or_null ? d_bias_or_null[i] : nullptr;
        const int relu = last ? relu_last : relu_hidden;
        float *out = last ? d_Y : (float *)region(act0, P.act_bytes, i);
        if (reads_xt(P.fc[i].path)) {
            // towards a following layer that takes its activations transposed, this layer's finishing
            // kernel writes them so, the image axis padded to that layer's tile
            const bool to_xt = !last && P.xt_in[i + 1];
            float *dst = to_xt ? (float *)region(xt0, P.xt_bytes, i + 1) : out;
            const int next_bp = !to_xt ? 0 : P.fc[i + 1].path == CL_PATH_SPARSE_WIDE ? P.fc[i + 1].wide.Bp : P.fc[i + 1].mfma.Bp;
            int32_t rc;
            if (P.fc[i].path == CL_PATH_SPARSE_WIDE)
                rc = run_wide_layer(L, D, P.fc[i].wide, in, (float *)region(xt0, P.xt_bytes, i), (float *)region(part0, P.part_bytes, i),
                                    ent_of(i), true, bias, dst, next_bp, batch, relu, st);
            else
                rc = run_mfma_layer(L, D, P.fc[i].mfma, in, region(xt0, P.xt_bytes, i), (float *)region(part0, P.part_bytes, i), bias, dst, next_bp, batch, relu, st);
            if (rc) return rc;
            in = to_xt ? nullptr : out;
        } else {
            // between two layers of this path at one image the finishing kernel is left out:
            // the next layer adds the partial tiles up as it stages its input
            PrevSlots prev{};
            if (P.fold_in[i]) {
                const cl_layer *Lp = layers[i - 1];
                prev = PrevSlots{(const float *)region(part0, P.part_bytes, i - 1), make_dev(Lp).panel_chunk,
                                 d_bias_or_null ? d_bias_or_null[i - 1] : nullptr, divisor((uint32_t)Lp->desc.block_h), P.fc[i - 1].sparse.wg_per_panel,
                                 batch, relu_hidden};
            }
            const bool finish = last || !P.fold_in[i + 1];
            if (int32_t rc = forward_sparse(L, D, P.fc[i].sparse, in, bias, out, batch, relu, (float *)region(part0, P.part_bytes, i), st,
                                            n_layers > 1, P.fold_in[i] ? &prev : nullptr, finish))
                return rc;
            in = out;
        }
    }
    clear_error();
    return CL_OK;
} catch (...) {
    return fail_with_exception();
}

// ------------------------------------------------------------------------- //
// several layers of one shape in one grid
// ------------------------------------------------------------------------- //
struct cl_layer_group {
    std::vector<const cl_layer *> layers;
    LayerDev *table = nullptr;        // device copy of the layers' LayerDev, in order
    int device = -1;
    int64_t max_panel_chunks = 0;     // over all layers
    size_t table_bytes = 0;           // largest table image (LDS) of any layer
    bool any_chunks = false;
};

namespace {

struct GroupPlan {
    SparsePlan sp;
    uint32_t wgs_per_layer = 0;
    size_t part_stride = 0;           // floats between the layers' partial tiles
    size_t lds = 0;
    int xcap = 0;
};

int32_t plan_group(const cl_layer_group *G, int batch, const DeviceLimits &dl, GroupPlan &P)
{
    const cl_layer *L = G->layers[0];
    if (batch < 1) return fail(CL_EINVAL, "batch must be positive");
    if (batch > 16 || (batch & (batch - 1))) return fail(CL_EUNSUPPORTED, "a group call takes 1, 2, 4, 8 or 16 images per layer");
    if (int32_t rc = plan_sparse(L, batch, dl, P.sp, true)) return rc;
    if (P.sp.bt_max < batch) return fail(CL_EUNSUPPORTED, "%d images do not fit one batch tile of this layer shape", batch);
    const int bt = batch;
    P.sp.bt_max = bt;
    P.sp.fixed = G->table_bytes;
    P.sp.wg_per_panel = (int)((G->max_panel_chunks + kWaves * kSparseChunksPerWave - 1) / (kWaves * kSparseChunksPerWave));
    P.wgs_per_layer = (uint32_t)std::max<int64_t>(1, (int64_t)L->n_panels * P.sp.wg_per_panel);
    P.part_stride = (size_t)P.wgs_per_layer * L->desc.block_h * bt;
    P.lds = P.sp.lds_for(L, bt);
    if (P.lds > dl.max_lds) return fail(CL_EUNSUPPORTED, "the layers' tables and a tile of %d images need more LDS than a workgroup has", bt);
    P.xcap = P.sp.xcap_for(bt);
    return CL_OK;
}

}  // namespace

extern "C" int32_t cl_layer_group_create(const cl_layer *const *layers, int32_t n_layers, cl_layer_group **out)
try {
    if (!layers || !out || n_layers < 1) return fail(CL_EINVAL, "a group needs at least one layer");
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    std::unique_ptr<cl_layer_group> G(new cl_layer_group());
    std::vector<LayerDev> host;
    for (int i = 0; i < n_layers; ++i) {
        const cl_layer *L = layers[i];
        if (int32_t rc = require_device(L)) return rc;
        const cl_layer *F = layers[0];
        if (L->desc.M != F->desc.M || L->desc.K != F->desc.K || L->desc.block_h != F->desc.block_h || L->desc.block_w != F->desc.block_w)
            return fail(CL_EINVAL, "layer %d differs from layer 0 in shape or block size", i);
        G->layers.push_back(L);
        host.push_back(make_dev(L));
        G->max_panel_chunks = std::max(G->max_panel_chunks, L->max_panel_chunks);
        G->table_bytes = std::max(G->table_bytes, table_image_bytes(L->val_lut_bits, L->idx_lut_bits, 1 << L->desc.weight_bits));
        G->any_chunks = G->any_chunks || L->n_chunks > 0;
    }
    G->device = dev;
    if (hipMalloc((void **)&G->table, host.size() * sizeof(LayerDev)) != hipSuccess)
        return fail(CL_ENOMEM, "hipMalloc of the group table failed");
    if (hipMemcpy(G->table, host.data(), host.size() * sizeof(LayerDev), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(G->table);
        return fail(CL_EHIP, "hipMemcpy of the group table failed");
    }
    *out = G.release();
    clear_error();
    return CL_OK;
} catch (...) {
    return fail_with_exception();
}

extern "C" void cl_layer_group_free(cl_layer_group *G)
{
    if (!G) return;
    if (G->table) (void)hipFree(G->table);
    delete G;
}

extern "C" int32_t cl_fc_group_workspace_bytes(const cl_layer_group *G, int32_t batch, size_t *out)
{
    if (!G || !out) return fail(CL_EINVAL, "null argument");
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    GroupPlan P;
    if (int32_t rc = plan_group(G, batch, dl, P)) return rc;
    *out = G->layers.size() * P.part_stride * sizeof(float);
    return CL_OK;
}

extern "C" int32_t cl_compressed_fc_group_forward(const cl_layer_group *G, const float *d_X, size_t x_stride,
                                                  const float *d_bias_or_null, size_t bias_stride, float *d_Y, int32_t batch,
                                                  int32_t relu, void *d_workspace, size_t workspace_bytes, void *stream)
{
    if (!G || !d_X || !d_Y) return fail(CL_EINVAL, "null argument");
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev != G->device) return fail(CL_EINVAL, "the group was created on device %d, the current device is %d", G->device, dev);
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    GroupPlan P;
    if (int32_t rc = plan_group(G, batch, dl, P)) return rc;
    const size_t n = G->layers.size(), need = n * P.part_stride * sizeof(float);
    if (workspace_bytes < need || !d_workspace) return fail(CL_EINVAL, "workspace too small: %zu < %zu", workspace_bytes, need);
    if ((uintptr_t)d_workspace % 256) return fail(CL_EINVAL, "workspace must be 256-byte aligned");
    const cl_layer *L = G->layers[0];
    hipStream_t st = (hipStream_t)stream;
    float *part = (float *)d_workspace;
    const int bt = P.sp.bt_max;
    if (G->any_chunks) {
        dim3 grid;
        GRID_TRY(grid, (int64_t)n * P.wgs_per_layer);
        timing_begin(st);
#define CL_LAUNCH_GROUP(BTV)                                                                                        \
    do {                                                                                                            \
        if (P.lds > 64 * 1024)                                                                                      \
            HIP_TRY(hipFuncSetAttribute((const void *)fc_sparse_group_kernel<BTV>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)P.lds)); \
        hipLaunchKernelGGL(fc_sparse_group_kernel<BTV>, grid, dim3(kThreads), P.lds, st, G->table, divisor(P.wgs_per_layer), d_X, x_stride, part, \
                           P.part_stride, divisor((uint32_t)P.sp.wg_per_panel), P.xcap);                                               \
    } while (0)
        switch (bt) {
        case 16: CL_LAUNCH_GROUP(16); break;
        case 8: CL_LAUNCH_GROUP(8); break;
        case 4: CL_LAUNCH_GROUP(4); break;
        case 2: CL_LAUNCH_GROUP(2); break;
        default: CL_LAUNCH_GROUP(1); break;
        }
#undef CL_LAUNCH_GROUP
        HIP_TRY(hipGetLastError());
        timing_end(st, 1);
    }
    const int red_per_layer = L->n_panels * bt;
    dim3 rgrid;
    GRID_TRY(rgrid, (int64_t)n * red_per_layer);
    hipLaunchKernelGGL(fc_reduce_group_kernel, rgrid, dim3(kRedThreads), 0, st, G->table, red_per_layer, part, P.part_stride,
                       d_bias_or_null, bias_stride, d_Y, (size_t)batch * L->desc.M, bt, P.sp.wg_per_panel, relu);
    HIP_TRY(hipGetLastError());
    clear_error();
    return CL_OK;
}

// ------------------------------------------------------------------------- //
// fixed-function layers of a whole network (Table IV: pool, norm)
// ------------------------------------------------------------------------- //

extern "C" int32_t cl_maxpool_forward(const float *d_X, float *d_Y, int32_t batch, int32_t C, int32_t H, int32_t W,
                                      int32_t size, int32_t stride, void *stream)
{
    if (!d_X || !d_Y) return fail(CL_EINVAL, "null pointer");
    if (batch < 1 || C < 1 || size < 1 || stride < 1 || H < size || W < size) return fail(CL_EINVAL, "bad pooling geometry");
    const int P = (H - size) / stride + 1, Q = (W - size) / stride + 1;
    if ((int64_t)P * Q > (1 << 30)) return fail(CL_EUNSUPPORTED, "more than 2^30 outputs per plane");
    const int64_t planes = (int64_t)batch * C;
    const int pq = P * Q, planes_per_row = (int)std::min<int64_t>(planes, std::max(1, 2048 / pq));
    const dim3 grid((unsigned)(((int64_t)planes_per_row * pq + 255) / 256),
                    (unsigned)std::min<int64_t>((planes + planes_per_row - 1) / planes_per_row, 65535));
    auto kernel = size == 3 ? maxpool_kernel<3> : size == 2 ? maxpool_kernel<2> : maxpool_kernel<0>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, (hipStream_t)stream, d_X, d_Y, planes, H, W, P, Q, size, stride, planes_per_row);
    HIP_TRY(hipGetLastError());
    clear_error();
    return CL_OK;
}

extern "C" int32_t cl_lrn_forward(const float *d_X, float *d_Y, int32_t batch, int32_t C, int32_t H, int32_t W,
                                  int32_t n, float alpha, float beta, float k, void *stream)
{
    if (!d_X || !d_Y) return fail(CL_EINVAL, "null pointer");
    if (batch < 1 || C < 1 || H < 1 || W < 1 || n < 1 || !(n & 1)) return fail(CL_EINVAL, "bad normalisation geometry");
    const int64_t hw = (int64_t)H * W, runs = (int64_t)batch * ((C + kLrnChunk - 1) / kLrnChunk);
    if (runs > INT32_MAX) return fail(CL_EUNSUPPORTED, "batch x channels too large");
    const dim3 grid((unsigned)((hw + 255) / 256), (unsigned)std::min<int64_t>(runs, 65535));
    const float a_n = alpha / (float)n;
    switch (n / 2) {
    case 1: hipLaunchKernelGGL(lrn_kernel<1>, grid, dim3(256), 0, (hipStream_t)stream, d_X, d_Y, batch, C, hw, n, a_n, beta, k); break;
    case 2: hipLaunchKernelGGL(lrn_kernel<2>, grid, dim3(256), 0, (hipStream_t)stream, d_X, d_Y, batch, C, hw, n, a_n, beta, k); break;
    default: hipLaunchKernelGGL(lrn_kernel<-1>, grid, dim3(256), 0, (hipStream_t)stream, d_X, d_Y, batch, C, hw, n, a_n, beta, k); break;
    }
    HIP_TRY(hipGetLastError());
    clear_error();
    return CL_OK;
}

extern "C" int32_t cl_set_kernel_timing(int32_t enable)
{
    if (enable && !g_timing.a) {
        HIP_TRY(hipEventCreate(&g_timing.a));
        HIP_TRY(hipEventCreate(&g_timing.b));
    }
    g_timing.on = enable != 0;
    g_timing.valid = false;
    return CL_OK;
}

extern "C" int32_t cl_last_kernel_ms(float *ms, int32_t *launches)
{
    if (!ms || !launches) return fail(CL_EINVAL, "null argument");
    if (!g_timing.on || !g_timing.valid) return fail(CL_EINVAL, "no timed forward call yet");
    HIP_TRY(hipEventSynchronize(g_timing.b));
    HIP_TRY(hipEventElapsedTime(ms, g_timing.a, g_timing.b));
    *launches = g_timing.launches;
    return CL_OK;
}

namespace {

// Launch shape of the convolution path: the batch is cut into groups of images whose
// column matrices (one per filter group) stay under kConvXtCap bytes; each group of
// images is one launch of the MFMA path over the block rows of all filter groups.
constexpr size_t kConvXtCap = (size_t)1024 << 20;

struct ConvPlan {
    ConvGeom cg{};
    int OCg = 0, panels_per_group = 0, imgs = 0;
    bool gather = false;       // blocks decoded once per call, no column matrix in memory: conv_mfma_kernel
    bool planes = false;       // operands split once per call: conv_plane_kernel
    PlaneGeom pg{};
    int tile = 0;              // its tile, the same for all image groups (the order of the split weights)
    int groups_at_once = 1;    // filter groups per launch: all of them, or one (the compact form)
    size_t lds = 0, xt_bytes = 0, part_bytes = 0, wt_bytes = 0, rows_bytes = 0;
    size_t total() const { return xt_bytes + part_bytes + wt_bytes + rows_bytes; }
};

// The shapes of conv_plane_kernel's workgroup tile.
struct PlaneTile {
    int rows, cols, mfmas;     // of a tile; accumulators of a wavefront
};
constexpr PlaneTile kPlaneTiles[3] = {{128, 128, 4}, {96, 128, 3}, {64, 128, 2}};

constexpr int kPlaneRun = 256;

// Split activations and partial tiles of a launch together: the images of a call are taken in groups that stay below this (one
// image at least), weights split with the first.  (VGG-16 conv1_2 at 64 images, 1.26 GB at once: us in 2 / 5 / 11 / 22 groups 1786 / 1796 / 1777 /
// 1880; conv2_2 in 1 / 3 / 5 / 11 1393 / 1444 / 1378 / 1568.  Of 8600 drawn fp32 calls that take the form eight are slower by more than 5 % with this limit than
// without any, and 137 with half of it.)
constexpr size_t kPlaneScratch = (size_t)256 << 20;

struct PlaneShape {
    int tile = 0, tiles = 0, splits = 1;
    int64_t cost = 0;          // cycles
};

// Tile and split of the steps of k by a model of the launch, in cycles: a step is a wavefront's multiplies and a quarter more (32 x 32 x 16
// multiplies take 32 cycles; with one workgroup to a CU 1.07 times that is measured, with two the chip's clock gives way), 5 k for a workgroup
// alone on its CU to start and end and 8 k for two; the partial tiles of split steps as in mfma_shape, 300 for a split's turn in the
// finishing launch and 8 k for that launch.  Over 230 drawn convolutions the launch takes 4 us + 1.11 times its price, and the tile picked is within 2 % of
// the best of the three on average, 13 % at worst.  (only: this tile, not the best of the three.)
PlaneShape plane_shape(int OCg, int groups, int steps, int ncols, bool bf16, int cus, int only = -1)
{
    cus = std::max(1, cus);
    PlaneShape best;
    for (int i = 0; i < 3; ++i) {
        if (only >= 0 && i != only) continue;
        const PlaneTile &T = kPlaneTiles[i];
        const int64_t panels = (int64_t)groups * ((OCg + T.rows - 1) / T.rows), tiles = (ncols + T.cols - 1) / T.cols;
        const int64_t step = (int64_t)(bf16 ? 3 : 8) * 32 * T.mfmas * 5 / 4;
        const int sp_max = (int)std::max<int64_t>(1, std::min<int64_t>(steps, (4 * cus + panels * tiles - 1) / (panels * tiles)));
        // (not more than kPlaneRun steps in one sum, which rounds at every one of them)
        for (int sp = (steps + kPlaneRun - 1) / kPlaneRun; sp <= std::max(sp_max, (steps + kPlaneRun - 1) / kPlaneRun);) {
            const int64_t items = panels * tiles * sp, n = (steps + sp - 1) / sp;
            const int64_t full = items / (2 * cus), rest = items % (2 * cus);
            int64_t t = full * (8000 + 2 * step * n);
            if (rest) t += rest <= cus ? 5000 + step * n : 8000 + 2 * step * n;
            if (sp > 1) t += 8000 + 300 * sp + panels * T.rows * tiles * T.cols * sp * 4 * 2 / 5000;
            if (best.cost == 0 || t < best.cost) best = PlaneShape{i, (int)tiles, sp, t};
            if (n == 1) break;
            sp = (int)((steps + n - 2) / (n - 1));          // the next that makes a workgroup's run of steps shorter
        }
    }
    return best;
}

// From this many columns on (image x output pixel) both paths decode the layer's
// blocks once per call into dense tiles in the workspace, and a multiply kernel of its own
// gathers each 128 x 128 piece of the column matrix into LDS straight from the input, so
// that the column matrix never exists in memory.  Below, and for calls too small to
// give that kernel's one tile width enough work items (see plan_conv), the column matrix
// is written out and the blocks of a column tile are decoded inside the multiply kernel
// (measured on the AlexNet and VGG-16 convolutions at 1 to 64 images: with these limits
// the gathered form is the faster one wherever it is taken, by 4-25 %; of thirty convolutions with 96 to
// 700 columns none gains more than 1 % from a limit of 96, one of 169 columns goes from 19.9 to 24.4 us).
constexpr int64_t kConvGatherColumns = 512;

// Whether the layer's weights are the sums of the three bf16 terms that the gathered form splits them
// into, with a sign that the first two share (split_weights): not below 2^-110, nor as -0.
bool splits_exactly(const cl_layer *L, float least = 0x1p-110f)
{
    for (float c : L->codebook)
        if (std::fabs(c) < least && (c != 0.0f || std::signbit(c))) return false;
    return true;
}

// Blocks side by side that a workgroup of conv_prepare_kernel decodes, fewer rows of each the more there are: enough that most of their
// units of eight channels are whole (162 channels of 11 x 11, us beside the multiply launch, 1 / 2 / 4 / 8 blocks: 109 / 77 / 67 / 69;
// VGG-16 conv4_2, 3 x 3: 25.1 / 24.4 / 26.2 / 29.5; 1 x 1: 8.3 / 8.8 / 8.7 / 8.9).
int prep_blocks(const cl_layer *L, int taps)
{
    const int most = taps == 1 ? 1 : taps < 16 ? 2 : 4;
    int n = 1;
    while (n < most && n < L->nbw) n *= 2;
    return n;
}

int64_t prep_strips(const cl_layer *L, int blocks)
{
    const int rows = kPrepCells / blocks;
    return (int64_t)L->n_panels * ((L->desc.block_h + rows - 1) / rows) * ((L->nbw + blocks - 1) / blocks);
}

// What a call of that form takes, in us: the call; each launch of a group of images; a CU's pair of workgroups, or one alone, to start and
// end, and a step of theirs by the tile; a MB of split weights, of filters of fewer than 16 taps and of others (which end more of their units in other workgroups); rounds of
// strips behind the first; a MB of split activations, of outputs, of partial tiles, the finishing launch and a split's turn in it; and, of
// strides above one, whose 64 pixels of a request lie that far apart, a MB requested (stride 2 by whether the terms of a launch exceed
// 90 MB, wider ones).  [bf16][four channels to a pixel], fitted to 32 k drawn calls of 25 us (bf16 18) and longer: 5.2 % off them (bf16 5.9 %).
struct PlanePrice {
    double call, run, pair, alone, step2[3], step1[3], weights[2], over, terms, outputs, part, split, turn, near, far, wide;
};
constexpr PlanePrice kPlanePrice[2][2] = {
    {{13.5, 25, 1.75, 2.2, {.599, .461, .299}, {.624, .485, .309}, {.97, 1.18}, 3.6, .17, .209, .23, 3.8, .124, .006, .023, .025},
     {12.2, 7, 2.9, 3.15, {.628, .477, .284}, {.644, .489, .309}, {2.65, 2.65}, 0, .20, .119, .73, .26, 0, .003, .003, .008}},
    {{14.5, 25, .05, 0, {.238, .196, .124}, {.285, .257, .210}, {1.07, 1.50}, 3.6, .216, .200, .31, 2.4, .163, .003, .052, .026},
     {13, 7, 1.17, 0, {.238, .200, .109}, {.326, .321, .251}, {3.5, 3.5}, 0, .15, .154, 0, 0, 0, .010, .010, .027}}};

// The form whose operands are split beforehand: its geometry and workspace, and what the call will take, in us; false where it cannot run.
bool plan_planes(const cl_layer *L, const cl_conv_desc *cv, int batch, bool bf16, const DeviceLimits &dl, ConvPlan &P, double &us)
{
    const ConvGeom &g = P.cg;
    const int np = bf16 ? 2 : 3;
    PlaneGeom &q = P.pg;
    q.C = g.C; q.Cg = g.Cg; q.H = g.H; q.W = g.W; q.R = g.R; q.S = g.S; q.pad = g.pad;
    q.px4 = g.Cg <= 4 ? 1 : 0;
    if (q.px4 && g.S < 2) return false;
    // (half a weight has to split, too, where two units share a tap)
    if (!bf16 && !splits_exactly(L, q.px4 && (g.S & 1) ? 0x1p-109f : 0x1p-110f)) return false;
    const int64_t Hp = g.H + 2 * (int64_t)g.pad, Wp = (g.W + 2 * (int64_t)g.pad + q.px4) / (1 + q.px4) * (1 + q.px4);
    q.CG = q.px4 ? 1 : (g.Cg + 7) / 8;
    q.SU = q.px4 ? (g.S + 1) / 2 : g.S;
    q.groups = cv->groups;
    q.OCg = P.OCg;
    // offsets are 32-bit ones: of the activations in bytes, all terms, and of a tile's weights
    const int64_t units = (int64_t)q.CG * g.R * q.SU;
    if (Hp > INT32_MAX / Wp || Hp * Wp > INT32_MAX / 16 / np / q.groups / q.CG || units > INT32_MAX / 2 / (np * kTile * 16)) return false;
    q.Hp = (int)Hp;
    q.Wp = (int)Wp;
    const int64_t plane = Hp * Wp / (1 + q.px4), image = (int64_t)q.groups * q.CG * plane;                // 16-byte pieces
    q.units = (int)units;
    q.steps = (q.units + 1) / 2;
    const int pq = g.P * g.Q;
    auto panels_of = [&](int tile) { return q.groups * ((P.OCg + kPlaneTiles[tile].rows - 1) / kPlaneTiles[tile].rows); };
    auto xs_of = [&](int imgs) { return round256((size_t)np * 16 * imgs * image); };
    auto part_of = [&](const PlaneShape &s) {
        const PlaneTile &T = kPlaneTiles[s.tile];
        return s.splits == 1 ? 0 : round256((size_t)panels_of(s.tile) * T.rows * s.splits * s.tiles * T.cols * sizeof(float));
    };
    // groups of equal size, as few as the launch's offsets and kPlaneScratch allow
    int most = (int)std::min<int64_t>({(int64_t)batch, kMaxTileColumns / pq, INT32_MAX / (image * 16 * np), std::max<int64_t>(1, kPlaneScratch / (image * 16 * np))});
    PlaneShape s;
    for (;;) {
        const int runs = (batch + most - 1) / most;
        P.imgs = (batch + runs - 1) / runs;
        s = plane_shape(P.OCg, q.groups, q.steps, P.imgs * pq, bf16, dl.cus);
        const size_t bytes = xs_of(P.imgs) + part_of(s);
        if (bytes <= kPlaneScratch || P.imgs == 1) break;
        most = std::max(1, std::min(P.imgs - 1, (int)(P.imgs * (double)kPlaneScratch / bytes)));
    }
    P.tile = s.tile;
    q.pieces = (uint32_t)(P.imgs * image);
    q.per_plane = divisor((uint32_t)plane);
    q.per_row = divisor((uint32_t)(Wp / (1 + q.px4)));
    q.planes = divisor((uint32_t)(q.groups * q.CG));
    q.per_s = divisor((uint32_t)g.S);
    q.per_group = divisor((uint32_t)(q.px4 ? q.SU : g.R * g.S));
    const size_t wt = (size_t)panels_of(P.tile) * kPlaneTiles[P.tile].rows * q.steps * np * 2 * 16;
    P.xt_bytes = xs_of(P.imgs);
    P.wt_bytes = round256(wt);
    P.part_bytes = part_of(s);
    const int blocks = prep_blocks(L, g.R * g.S);
    const int64_t strips = prep_strips(L, blocks);
    if (strips > UINT32_MAX / kPrepThreads - 1024) return false;             // (a launch's threads are counted in 32 bits)
    const int cus = std::max(1, dl.cus);
    const PlanePrice &p = kPlanePrice[bf16][q.px4];
    us = p.call - p.run + p.weights[g.R * g.S >= 16] * 1e-6 * cv->out_channels * q.steps * np * 2 * 16 + p.over * std::max(0.0, (double)strips / cus - 1);
    for (int imgs : {P.imgs, batch % P.imgs}) {
        if (imgs == 0) continue;
        if (imgs != P.imgs) {
            s = plane_shape(P.OCg, q.groups, q.steps, imgs * pq, bf16, dl.cus, P.tile);
            P.part_bytes = std::max(P.part_bytes, part_of(s));
        }
        const int panels = panels_of(P.tile), n = (q.steps + s.splits - 1) / s.splits;
        const int64_t items = (int64_t)panels * s.tiles * s.splits, rest = items % (2 * cus);
        const int64_t pairs = items / (2 * cus) + (rest > cus ? 1 : 0);
        const double xs = 1e-6 * np * 16 * imgs * image, out = 4e-6 * imgs * cv->out_channels * pq;
        const double fetched = 1e-6 * np * 16 * 2 * q.steps * panels * imgs * pq;
        double t = p.run + pairs * (p.pair + 2 * n * p.step2[P.tile]) + (rest > 0 && rest <= cus ? p.alone + n * p.step1[P.tile] : 0) +
                   p.terms * xs + p.outputs * out;
        if (s.splits > 1) t += p.split + p.turn * (s.splits - 1) + p.part * 1e-6 * part_of(s);
        if (g.stride > 2) t += p.wide * fetched;
        else if (g.stride == 2) t += (xs > 90 ? p.far : p.near) * fetched;
        us += (imgs == P.imgs ? batch / P.imgs : 1) * t;
    }
    P.rows_bytes = round256((size_t)q.steps * 2 * sizeof(uint32_t));
    P.lds = table_image_bytes(L->val_lut_bits, L->idx_lut_bits, 1 << L->desc.weight_bits) + prep_tile_bytes(blocks) + ((size_t)2 * sizeof(uint2) << L->desc.weight_bits);
    return P.lds <= dl.max_lds;
}

// What a call of the other two forms takes, in us: the call; a workgroup's item (without a column matrix) or a cycle of mfma_shape's price (with
// one); a 64-wide half of a block, by the blocks' height in thirty-twos (with a column matrix: a block of a row's share); a MB of decoded blocks, of column matrix, of
// inputs, of outputs; the finishing launch and a MB of partial tiles where block rows are split.  Fitted to the same calls as PlanePrice:
// 6 % off them (bf16 8 %).  [bf16][filters of up to 32 taps] and [bf16].
struct OtherPrice {
    double call, item, half[4], weights, columns, inputs, outputs, split, part;
};
constexpr OtherPrice kGatherPrice[2][2] = {
    {{12.3, .9, {1.91, 2.20, 2.71, 2.87}, .54, 0, .57, .44, 4.4, .45}, {14, 1.3, {1.71, 1.93, 2.75, 2.88}, .50, 0, .09, .25, 2.6, .385}},
    {{12.7, .65, {1.19, 1.35, 1.55, 1.62}, .67, 0, .78, .35, 2.4, .56}, {11.7, 1.4, {1.03, 1.17, 1.54, 1.59}, .79, 0, .16, .23, 2.2, .46}}};
constexpr OtherPrice kColumnsPrice[2] = {{7.1, 1.13, {1.2}, 0, .28, 0, .35, 3.1, .23}, {4.7, 1.33, {0}, 0, .58, 0, 1.7, 0, .53}};

// any: whichever is the fastest.  not_planes: operands not split beforehand, which takes less scratch.  compact: the form that needs the
// least - filter groups one after the other through the same buffers, blocks decoded inside the multiply kernel.
enum class ConvForm { any, not_planes, compact };

int32_t plan_conv(const cl_layer *L, const cl_conv_desc *cv, int batch, bool bf16, const DeviceLimits &dl, ConvPlan &P,
                  ConvForm form = ConvForm::any)
{
    const bool compact = form == ConvForm::compact;
    if (!cv) return fail(CL_EINVAL, "null convolution descriptor");
    if (cv->C < 1 || cv->H < 1 || cv->W < 1 || cv->R < 1 || cv->S < 1 || cv->stride < 1 || cv->pad < 0 || cv->groups < 1 ||
        cv->out_channels < 1)
        return fail(CL_EINVAL, "bad convolution geometry");
    if (cv->C % cv->groups || cv->out_channels % cv->groups) return fail(CL_EINVAL, "groups must divide C and out_channels");
    ConvGeom &g = P.cg;
    g.C = cv->C; g.H = cv->H; g.W = cv->W; g.R = cv->R; g.S = cv->S; g.stride = cv->stride; g.pad = cv->pad;
    g.Cg = cv->C / cv->groups;
    g.P = (cv->H + 2 * cv->pad - cv->R) / cv->stride + 1;
    g.Q = (cv->W + 2 * cv->pad - cv->S) / cv->stride + 1;
    if (g.P < 1 || g.Q < 1) return fail(CL_EINVAL, "filter larger than the padded input");
    if ((int64_t)cv->H * cv->W > INT32_MAX / 2 || (int64_t)g.P * g.Q > kMaxTileColumns || (int64_t)g.Cg * g.R * g.S > INT32_MAX / 2)
        return fail(CL_EUNSUPPORTED, "image planes of more than 2^30 pixels or %d output pixels are not supported", kMaxTileColumns);
    if (L->desc.M != cv->out_channels || L->desc.K != g.Cg * g.R * g.S)
        return fail(CL_EINVAL, "layer is %d x %d, the convolution needs %d x %d", L->desc.M, L->desc.K, cv->out_channels, g.Cg * g.R * g.S);
    if (!mfma_capable(L)) return fail(CL_EUNSUPPORTED, "the convolution path needs blocks of at most %d x %d", kTile, kTile);
    P.OCg = cv->out_channels / cv->groups;
    if (cv->groups > 1 && P.OCg % L->desc.block_h) return fail(CL_EUNSUPPORTED, "block_h %d must divide the %d filters of a group", L->desc.block_h, P.OCg);
    P.panels_per_group = (P.OCg + L->desc.block_h - 1) / L->desc.block_h;
    P.groups_at_once = compact ? 1 : cv->groups;
    const int launch_panels = P.panels_per_group * P.groups_at_once;
    const size_t per_image = (size_t)P.groups_at_once * xt_rows(L) * g.P * g.Q * sizeof(float);
    P.imgs = (int)std::max<size_t>(1, std::min<size_t>((size_t)batch, kConvXtCap / per_image));
    P.lds = mfma_lds_bytes(L, bf16);
    if (P.lds > dl.max_lds) return fail(CL_EUNSUPPORTED, "the convolution path needs %zu bytes of LDS", P.lds);
    const int64_t cols = (int64_t)batch * g.P * g.Q;
    const int planes = bf16 ? 2 : 3;
    P.gather = !compact && cols >= kConvGatherColumns && (size_t)conv_lds_bytes(planes) <= dl.max_lds &&
               // its one tile width must give the chip something to do: work items for a
               // sixteenth of the CUs before the block rows are split, 128 x 128 products for half
               16 * launch_panels * ((cols + kConvColumns - 1) / kConvColumns) >= dl.cus &&
               2 * launch_panels * ((cols + kConvColumns - 1) / kConvColumns) * L->nbw >= dl.cus &&
               (int64_t)(kConvColumns + 1) * g.C * g.H * g.W < (1 << 29) && g.R <= 32 && g.S <= 32 &&    // the gatherers' 32-bit byte offsets and tap masks
               (bf16 || splits_exactly(L));
    if (P.gather) {
        // nothing but the launch size limits the images of a launch
        P.imgs = (int)std::min<int64_t>(batch, kMaxTileColumns / ((int64_t)g.P * g.Q));
        P.lds = (size_t)conv_lds_bytes(planes);
    }
    P.wt_bytes = P.gather ? (size_t)L->n_blocks * kTile * kTile * sizeof(float) : 0;
    P.rows_bytes = P.gather ? round256((size_t)L->nbw * kTile * sizeof(uint2)) : 0;
    // workspace for the larger of a full image group and the last, smaller one
    P.xt_bytes = P.part_bytes = 0;
    double us = 0, cycles = 0;                              // what the call will take, to be compared with plan_planes'; mfma_shape's price
    const OtherPrice &p = P.gather ? kGatherPrice[bf16][g.R * g.S <= 32] : kColumnsPrice[bf16];
    const int nh = conv_halves(L->desc.block_w), height = std::min(3, (L->desc.block_h - 1) / 32);
    for (int imgs : {P.imgs, batch % P.imgs}) {
        if (imgs == 0) continue;
        int nq, np, splits;
        int64_t cost;
        mfma_shape(L, launch_panels, imgs * g.P * g.Q, dl.cus, bf16, nq, np, splits, P.gather, P.gather || !bf16, &cost);
        const size_t xt = P.gather ? 0 : (size_t)P.groups_at_once * xt_bytes_for(L, np, bf16);
        const size_t part = (size_t)launch_panels * splits * np * L->desc.block_h * sizeof(float);
        double t = p.columns * 1e-6 * xt + 4e-6 * imgs * ((double)p.inputs * g.C * g.H * g.W + p.outputs * cv->out_channels * g.P * g.Q);
        if (splits > 1) t += p.split + p.part * 1e-6 * part;
        if (P.gather) {
            const int rounds = (int)(((int64_t)launch_panels * splits * (np / kConvColumns) + std::max(1, dl.cus) - 1) / std::max(1, dl.cus));
            const int halves = splits > 1 ? (L->nbw + splits - 1) / splits * nh
                                          : (L->nbw - 1) * nh + conv_halves(L->desc.K - (L->nbw - 1) * L->desc.block_w);
            t += rounds * (p.item + halves * p.half[height]);
        } else t += p.item * cost / 2400 + p.half[0] * L->nbw / splits;
        const int runs = imgs == P.imgs ? batch / P.imgs : 1;
        us += runs * t;
        cycles += runs * (double)cost;
        P.xt_bytes = std::max(P.xt_bytes, xt);
        if (!(P.gather && splits == 1)) P.part_bytes = std::max(P.part_bytes, part);
    }
    us += p.call + p.weights * 1e-6 * P.wt_bytes;
    // Both operands split beforehand, where that is cheaper by a twenty-fifth and the call a long one.  What it saves is in proportion to
    // the multiplies, what it costs to the weights (VGG-16 conv4_2 at one image, 14 MB of terms: 19 us to split them and 30 to multiply, gathered 9
    // and 36).  Of 14200 fp32 calls drawn anew 6250 take it, 1.30 times as fast on average as the other two forms, 0.3 % of them slower by more than 5 % (14 % at
    // worst); of 4800 bf16 ones 3330, 1.37 times, 0.8 % slower (23 %).  (With one price for all of a form's calls, without launches that add up, strides and
    // halves of blocks, 0.7 % and 6 % were, up to 27 % and 59 %, and AlexNet's conv1 and conv5 at 64 images, 1.25 and 1.08 times as fast in this form, did not take it.)
    // Long: some 36 us by mfma_shape's price, below which several times the scratch would buy some 8 %; in bf16, 17 us, below which there is nothing to gain.
    const bool long_call = bf16 ? us > 17 : P.gather ? 1.11 * cycles / 2400 + 1.1e-6 * P.wt_bytes > 21.5 : 2.1 * cycles / 2400 > 36;
    if (form == ConvForm::any && long_call) {
        ConvPlan F = P;
        double planes_us;
        if (plan_planes(L, cv, batch, bf16, dl, F, planes_us) && 1.04 * planes_us < us) {
            P = F;
            P.planes = true;
        }
    }
    return CL_OK;
}

}  // namespace

static int32_t conv_scratch(const cl_layer *L, const cl_conv_desc *cv, int32_t batch, int32_t path, size_t *out, std::initializer_list<ConvForm> forms)
{
    if (!L || !out) return fail(CL_EINVAL, "null argument");
    if (batch < 1) return fail(CL_EINVAL, "batch must be positive");
    if (path != CL_PATH_AUTO && !is_mfma(path)) return fail(CL_EUNSUPPORTED, "convolution runs on the MFMA paths only");
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    size_t least = SIZE_MAX;
    for (ConvForm form : forms) {
        ConvPlan P;
        if (int32_t rc = plan_conv(L, cv, batch, path == CL_PATH_MFMA_BF16, dl, P, form)) return rc;
        least = std::min(least, P.total());
    }
    *out = least;
    return CL_OK;
}

extern "C" int32_t cl_conv_workspace_bytes(const cl_layer *L, const cl_conv_desc *cv, int32_t batch, int32_t path, size_t *out)
{
    return conv_scratch(L, cv, batch, path, out, {ConvForm::any});
}

extern "C" int32_t cl_conv_workspace_bytes_unsplit(const cl_layer *L, const cl_conv_desc *cv, int32_t batch, int32_t path, size_t *out)
{
    return conv_scratch(L, cv, batch, path, out, {ConvForm::not_planes});
}

// (the faster forms' launch shapes can happen to need less than the compact one's)
extern "C" int32_t cl_conv_workspace_bytes_min(const cl_layer *L, const cl_conv_desc *cv, int32_t batch, int32_t path, size_t *out)
{
    return conv_scratch(L, cv, batch, path, out, {ConvForm::compact, ConvForm::any, ConvForm::not_planes});
}

namespace {

// One group of images of a convolution call: what the forms share.
struct ConvCall {
    const cl_layer *L;
    const ConvPlan *P;
    LayerDev D;
    const float *x;         // the group's input, images x C x H x W
    float *y;               // its output, images x M x pq
    const float *bias;
    int ncols, pq, relu;    // columns = images x output pixels
    int launch_panels, nq, Np, splits;
    float *part;
    hipStream_t st;
    int cus;
    bool *timed;            // benchmarks time the first multiply launch of a call
};

// adds the splits of the block rows, bias, activation, NCHW
int32_t conv_finish_splits(const ConvCall &c)
{
    const int ct = reduce_col_tile(c.launch_panels, c.ncols);
    dim3 grid;
    GRID_TRY(grid, (int64_t)c.launch_panels * ((c.ncols + ct - 1) / ct));
    hipLaunchKernelGGL(mfma_reduce_kernel, grid, dim3(256), 0, c.st,
                       c.D, c.part, c.bias, c.y, c.ncols, c.Np, c.splits, c.relu, c.pq, ct, 0, c.L->desc.block_h);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

// The gathered form: one launch gathers the columns and multiplies them with the decoded
// blocks (wt) of all filter groups; it finishes the output itself unless block rows are split.
int32_t conv_gathered(const ConvCall &c, bool bf16, const float *wt, const uint2 *rows, bool combined)
{
    const ConvPlan &P = *c.P;
    const bool direct = c.splits == 1;
    // (partial tiles take neither bias nor activation)
    const DirectOut out{direct ? c.y : nullptr, direct ? c.bias : nullptr, c.ncols, c.pq, direct ? c.relu : 0};
    // the kernel form for the height of the layer's blocks: how the multiplying wavefronts divide the tile
    const int bh = c.L->desc.block_h;
    using Kernel = void (*)(LayerDev, const float *, const float *, const uint2 *, float *, ConvGeom, int, int, int, int, int, DirectOut);
    static const Kernel kernels[8] = {conv_mfma_kernel<false, 4, 3>, conv_mfma_kernel<true, 4, 3>, conv_mfma_kernel<false, 2, 3>, conv_mfma_kernel<true, 2, 3>,
                                      conv_mfma_kernel<false, 4, 2>, conv_mfma_kernel<true, 4, 2>, conv_mfma_kernel<false, 2, 2>, conv_mfma_kernel<true, 2, 2>};
    static LdsLimit seen[8];
    const int which = (combined ? 1 : 0) + (bh <= 64 ? 2 : 0) + (bf16 ? 4 : 0);
    if (int32_t rc = ensure_lds((const void *)kernels[which], P.lds, seen[which])) return rc;
    dim3 grid;
    const int64_t items = (int64_t)c.launch_panels * c.splits * (c.Np / kConvColumns);
    if (items > INT32_MAX / 2) return fail(CL_EUNSUPPORTED, "a launch of %lld work items does not fit a grid", (long long)items);
    GRID_TRY(grid, std::min<int64_t>(items, std::max(1, c.cus)));
    if (!*c.timed) timing_begin(c.st);
    hipLaunchKernelGGL(kernels[which], grid, dim3(conv_threads(bf16 ? 2 : 3)), P.lds, c.st, c.D, c.x, wt, rows, c.part, P.cg, c.ncols, c.Np, c.splits,
                       P.panels_per_group, (int)items, out);
    HIP_TRY(hipGetLastError());
    if (!*c.timed) { timing_end(c.st, 1); *c.timed = true; }
    if (direct) return CL_OK;
    GRID_TRY(grid, (int64_t)c.L->desc.M * ((c.ncols + kConvRedColumns - 1) / kConvRedColumns));
    hipLaunchKernelGGL(conv_reduce_kernel, grid, dim3(kConvRedThreads), 0, c.st, c.part, c.bias, c.y, c.L->desc.M, P.OCg, P.panels_per_group, bh, c.ncols,
                       c.Np, c.splits, c.relu, c.pq);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

template <int NP, int RT, int CT, int WR, int WC>
int32_t launch_plane(dim3 grid, const uint4 *wt, const uint4 *xs, const uint32_t *unit_off, float *part, const PlaneConv &pc, hipStream_t st)
{
    hipLaunchKernelGGL((conv_plane_kernel<NP, RT, CT, WR, WC>), grid, dim3(256), 0, st, wt, xs, unit_off, part, pc);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

// The form with both operands split beforehand: one launch to split them (of the first images the weights too), one to multiply, one
// to add up where the steps are split.
int32_t conv_planes(const ConvCall &c, bool bf16, int imgs, bool first, void *xs, void *wt, uint32_t *unit_off)
{
    const ConvPlan &P = *c.P;
    PlaneGeom g = P.pg;
    const PlaneShape s = plane_shape(P.OCg, g.groups, g.steps, c.ncols, bf16, c.cus, P.tile);
    const PlaneTile &T = kPlaneTiles[P.tile];
    g.tile_rows = T.rows;
    g.ppg = (P.OCg + T.rows - 1) / T.rows;
    const uint32_t image = g.planes.d * g.per_plane.d;
    g.pieces = (uint32_t)imgs * image;
    const int blocks = prep_blocks(c.L, P.cg.R * P.cg.S);
    const int64_t n_strips = first ? prep_strips(c.L, blocks) : 0;
    dim3 grid;
    // (few strips: several workgroups decode the same one and each writes some of its units)
    const int parts = first ? (int)std::max<int64_t>(1, std::min<int64_t>(8, std::max(1, c.cus) / n_strips)) : 1;
    GRID_TRY(grid, n_strips * parts + std::min<int64_t>(1024, (g.pieces + kPrepThreads - 1) / kPrepThreads));
    using Prepare = void (*)(LayerDev, PlaneGeom, const float *, uint4 *, uint4 *, uint32_t *, int, int, int);
    static const Prepare prepare[2] = {conv_prepare_kernel<3>, conv_prepare_kernel<2>};
    static LdsLimit seen[2];
    if (int32_t rc = ensure_lds((const void *)prepare[bf16], P.lds, seen[bf16])) return rc;
    hipLaunchKernelGGL(prepare[bf16], grid, dim3(kPrepThreads), P.lds, c.st, c.D, g, c.x, (uint4 *)wt, (uint4 *)xs, unit_off, (int)n_strips, parts, blocks);
    HIP_TRY(hipGetLastError());
    PlaneConv pc{};
    pc.steps = g.steps; pc.splits = s.splits; pc.panels = g.groups * g.ppg; pc.ppg = g.ppg; pc.tiles = s.tiles;
    pc.n_cols = c.ncols; pc.Np = s.tiles * T.cols; pc.pq = c.pq; pc.Q = P.cg.Q; pc.stride = P.cg.stride;
    pc.Wp = g.Wp; pc.px_bytes = g.px4 ? 8 : 16;
    pc.image_bytes = image * 16; pc.group_bytes = (uint32_t)g.CG * g.per_plane.d * 16; pc.term_bytes = g.pieces * 16;
    pc.M = c.L->desc.M; pc.OCg = P.OCg;
    const bool direct = s.splits == 1;
    pc.Y = direct ? c.y : nullptr; pc.bias = c.bias; pc.relu = c.relu;
    GRID_TRY(grid, (int64_t)pc.panels * pc.tiles * pc.splits);
    if (!*c.timed) timing_begin(c.st);
    const uint4 *w = (const uint4 *)wt, *x = (const uint4 *)xs;
    int32_t rc;
    switch (s.tile + (bf16 ? 3 : 0)) {
    case 0: rc = launch_plane<3, 2, 2, 2, 2>(grid, w, x, unit_off, c.part, pc, c.st); break;
    case 1: rc = launch_plane<3, 3, 1, 1, 4>(grid, w, x, unit_off, c.part, pc, c.st); break;
    case 2: rc = launch_plane<3, 2, 1, 1, 4>(grid, w, x, unit_off, c.part, pc, c.st); break;
    case 3: rc = launch_plane<2, 2, 2, 2, 2>(grid, w, x, unit_off, c.part, pc, c.st); break;
    case 4: rc = launch_plane<2, 3, 1, 1, 4>(grid, w, x, unit_off, c.part, pc, c.st); break;
    default: rc = launch_plane<2, 2, 1, 1, 4>(grid, w, x, unit_off, c.part, pc, c.st); break;
    }
    if (rc) return rc;
    if (!*c.timed) { timing_end(c.st, 1); *c.timed = true; }
    if (direct) return CL_OK;
    GRID_TRY(grid, (int64_t)pc.M * ((c.ncols + kConvRedColumns - 1) / kConvRedColumns));
    hipLaunchKernelGGL(conv_reduce_kernel, grid, dim3(kConvRedThreads), 0, c.st, c.part, c.bias, c.y, pc.M, P.OCg, g.ppg, T.rows, c.ncols, pc.Np, s.splits, c.relu, c.pq);
    HIP_TRY(hipGetLastError());
    return CL_OK;
}

// The form with the column matrix in memory: P.groups_at_once filter groups per launch of
// each kernel; group grp of a launch has its column matrix at xt + grp * x_bytes and
// multiplies its own block rows.
int32_t conv_columns(ConvCall c, int groups_total, bool bf16, void *xt)
{
    const ConvPlan &P = *c.P;
    const cl_layer *L = c.L;
    const size_t x_bytes = xt_bytes_for(L, c.Np, bf16);
    for (int grp0 = 0; grp0 < groups_total; grp0 += P.groups_at_once) {
        const unsigned groups = (unsigned)P.groups_at_once;
        c.D.panel0 = grp0 * P.panels_per_group;
        if (bf16)
            hipLaunchKernelGGL(im2col_split_kernel, dim3((unsigned)std::min((c.Np + 63) / 64, 4096), (unsigned)(L->nbw * 8), groups), dim3(256), 0,
                               c.st, c.x, (uint16_t *)xt, P.cg, x_bytes / sizeof(uint16_t), c.ncols, c.Np, L->desc.block_w, L->desc.K,
                               xb_plane_elems(L, c.Np), grp0);
        else {
            // rows per workgroup: as many (up to kIm2colRows) as leave a couple of thousand workgroups
            const int64_t col_wgs = std::min((c.Np / 4 + 255) / 256, 4096);
            int rpw = kIm2colRows;
            while (rpw > 1 && col_wgs * (L->nbw * kTile / rpw) * groups < 2048) rpw >>= 1;
            hipLaunchKernelGGL(im2col_pad_kernel, dim3((unsigned)col_wgs, (unsigned)(L->nbw * kTile / rpw), groups), dim3(256), 0, c.st,
                               c.x, (float *)xt, P.cg, x_bytes / sizeof(float), c.ncols, c.Np, L->desc.block_w, L->desc.K, grp0, rpw);
        }
        HIP_TRY(hipGetLastError());
        if (!*c.timed) timing_begin(c.st);
        // block rows that are not split need no adding up: the multiply kernel finishes the output
        const bool direct = !bf16 && c.splits == 1;
        const DirectOut out{direct ? c.y : nullptr, c.bias, c.ncols, c.pq, c.relu};
        if (int32_t rc = launch_mfma(L, c.D, bf16, c.nq, c.launch_panels, c.splits, c.Np, P.panels_per_group, x_bytes, P.lds, xt, c.part, c.st, out))
            return rc;
        if (!*c.timed) { timing_end(c.st, 1); *c.timed = true; }
        if (!direct)
            if (int32_t rc = conv_finish_splits(c)) return rc;
    }
    return CL_OK;
}

}  // namespace

extern "C" int32_t cl_compressed_conv_forward(const cl_layer *L, const cl_conv_desc *cv, const float *d_X,
                                              const float *d_bias, float *d_Y, int32_t batch, int32_t relu,
                                              int32_t path, void *d_workspace, size_t workspace_bytes, void *stream)
{
    if (int32_t rc = require_device(L)) return rc;
    if (!d_X || !d_Y) return fail(CL_EINVAL, "null activation pointer");
    if (batch < 1) return fail(CL_EINVAL, "batch must be positive");
    if (path != CL_PATH_AUTO && !is_mfma(path)) return fail(CL_EUNSUPPORTED, "convolution runs on the MFMA paths only");
    if ((uintptr_t)d_workspace % 256) return fail(CL_EINVAL, "workspace must be 256-byte aligned");
    DeviceLimits dl;
    if (int32_t rc = device_limits(dl)) return rc;
    const bool bf16 = path == CL_PATH_MFMA_BF16;
    // the fast form if the workspace holds it, then the gathered one, else the compact one
    ConvPlan P;
    if (int32_t rc = plan_conv(L, cv, batch, bf16, dl, P)) return rc;
    const size_t fast = P.total();
    if (P.planes && (workspace_bytes < fast || !d_workspace)) {
        P = ConvPlan{};
        if (int32_t rc = plan_conv(L, cv, batch, bf16, dl, P, ConvForm::not_planes)) return rc;
    }
    if (workspace_bytes < P.total() || !d_workspace) {
        P = ConvPlan{};
        if (int32_t rc = plan_conv(L, cv, batch, bf16, dl, P, ConvForm::compact)) return rc;
        if (workspace_bytes < P.total() || !d_workspace)
            return fail(CL_EINVAL, "workspace too small: %zu < %zu (%zu for the fast form)", workspace_bytes, P.total(), fast);
    }
    hipStream_t st = (hipStream_t)stream;
    const ConvGeom &g = P.cg;
    // the workspace: column matrices (not in the gathered form), partial tiles, decoded blocks, row table
    char *ws = (char *)d_workspace;
    void *xt = ws;
    float *part = (float *)(ws + P.xt_bytes);
    float *wt = (float *)(ws + P.xt_bytes + P.part_bytes);
    uint2 *rows = (uint2 *)(ws + P.xt_bytes + P.part_bytes + P.wt_bytes);
    const bool combined = g.R * g.S <= 32;      // one tap mask per column instead of one per filter row and one per filter column
    if (P.gather && !P.planes) {
        const size_t lds = table_image_bytes(L->val_lut_bits, L->idx_lut_bits, 1 << L->desc.weight_bits) + (size_t)kWTileBytes;
        static LdsLimit seen;
        if (int32_t rc = ensure_lds((const void *)decode_tiles_kernel, lds, seen)) return rc;
        // n_blocks workgroups of kTileDecodeThreads threads: more threads than the row table has entries
        hipLaunchKernelGGL(decode_tiles_kernel, dim3((unsigned)L->n_blocks), dim3(kTileDecodeThreads), lds, st, make_dev(L), wt, g, L->nbw * kTile,
                           combined ? 1 : 0, rows);
        HIP_TRY(hipGetLastError());
    }
    bool timed = false;
    ConvCall c{L, &P, make_dev(L), nullptr, nullptr, d_bias, 0, g.P * g.Q, relu, P.panels_per_group * P.groups_at_once, 0, 0, 0, part, st, dl.cus, &timed};
    for (int b0 = 0; b0 < batch; b0 += P.imgs) {
        const int nb = std::min(P.imgs, batch - b0);
        c.ncols = nb * c.pq;
        c.x = d_X + (size_t)b0 * g.C * g.H * g.W;
        c.y = d_Y + (size_t)b0 * L->desc.M * c.pq;
        if (P.planes) {
            if (int32_t rc = conv_planes(c, bf16, nb, b0 == 0, xt, wt, (uint32_t *)rows)) return rc;
            continue;
        }
        mfma_shape(L, c.launch_panels, c.ncols, dl.cus, bf16, c.nq, c.Np, c.splits, P.gather, P.gather || !bf16);
        if (int32_t rc = P.gather ? conv_gathered(c, bf16, wt, rows, combined) : conv_columns(c, cv->groups, bf16, xt)) return rc;
    }
    clear_error();
    return CL_OK;
}
