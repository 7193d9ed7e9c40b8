// CD-SGD per-step data-parallel hot path for gfx950 (MI355X): the C ABI and the host side of every
// entry point.  One translation unit; the kernels are in the .hpp files beside this one:
//   tuning.hpp          build-time knobs (launch shapes, cache policy)
//   device_common.hpp   chunk geometry, 128-bit loads / stores, 16-bit widening, the quantiser
//   device_tables.hpp   extents, tensor descriptors, chunk table
//   kernels_tensor.hpp  single-tensor kernels (quantise-and-pack, update)
//   kernels_sparse.hpp  sparse form of a packed stream
//   decode_tile.hpp     decode-and-sum of one tile, all workers; decode-and-sum of one tensor
//   kernels_probe.hpp   bare streaming kernel (measurement aid)
//   kernels_fused.hpp   passes over a layer list: fused compressed pass, passes on 32-bit gradients
//   kernels_static.hpp  tables built on the device for the entry point that allocates nothing
//
// Work decomposition.  The unit of work of one lane is a "quad": four
// consecutive fp32 elements = one 128-bit load/store per buffer = one byte of
// the packed stream (four 2-bit codes; element e of a tensor is bits
// [2(e%4)+1 : 2(e%4)] of packed byte e/4, which is the little-endian view of
// the 32-bit-word layout in cdsgd.h).  A tensor is cut into "chunks" of 1024
// quads (4096 elements, 1 KiB of a packed stream); the chunk table of a plan
// lists (tensor, chunk) pairs, and only a tensor's last chunk can be ragged.
//   * The kernels over a layer list work on parts of a chunk, one quad per
//     lane: "tiles" of 256 lanes for the compressed pass (the peers' codes are
//     decoded word by word, decode_tile.hpp), "pieces" of one wave for the
//     passes on 32-bit gradients.
//   * Of the single-tensor kernels, decode-and-sum works in the same tiles,
//     one to four to a group, quantise-and-pack and the update in single-wave
//     pieces.
// Either way every wave instruction on an fp32 buffer touches one contiguous
// 1 KiB span: all traffic is fully coalesced.
//
// The path is elementwise and HBM-bound: no MFMA.  Each of grad / residual /
// w_global is read once and each of residual / w_global / w_local is written
// once per step.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "cdsgd.h"

#include "tuning.hpp"
#include "device_common.hpp"
#include "device_tables.hpp"
#include "kernels_tensor.hpp"
#include "kernels_sparse.hpp"
#include "decode_tile.hpp"
#include "kernels_probe.hpp"
#include "kernels_fused.hpp"
#include "kernels_static.hpp"

// The tables of cdsgd_step_fused_static live here (about 4.6 MiB on every GPU the library
// runs on, until the process ends).  In host code this name is only a handle for
// hipGetSymbolAddress; the device address is looked up once per device (static_scratch).
static __device__ __align__(256) unsigned char scratch[kStaticBytes];

namespace {

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// LDS that the single-wave kernels ask for at launch and never touch: it bounds the waves resident per
// compute unit (160 KiB / bytes).  With all 32 resident, more requests queue in front of HBM than it takes
// to keep it busy, and a mix of reads and writes is then served more slowly.  Measured (2^27 elements or the
// VGG-16-shaped list; TB/s at 32 / 26 / 22 / 20 / 17 / 16 / 13 / 10 resident waves):
//   correction pass with agg_full   6.42-6.45 / 6.40 / 6.51 / 6.66-6.67 / 6.55 / 6.55-6.60 / 6.41 / 5.88
//   quantise-and-pack               6.71 / 6.72 / - / 6.83 / - / 6.88 / 6.09 / 5.10
//   update, both rules              6.36 / 6.34 / - / 6.55 / - / 6.50 / 6.55 / 6.18
//   correction pass, sum in kernel  6.19 / 6.39-6.41 / 6.35 / 6.24 / - / 5.97   (by size and type: lds_of_kernel_sum)
// eq. 11 alone over a list loses with any bound and gets none; the single-tensor calls have theirs by length (small ones none);
// the compressed pass has a rule of its own (compressed_launch).
// The same bound stated to the compiler instead (amdgpu_waves_per_eu with a maximum of 5) gives 6.55 and 6.45 TB/s on
// the first and the third line: most of the gain, not all of it.  While a pass launched this way runs it holds the
// compute units' LDS, so a kernel of another stream that needs LDS waits for it; a full-gradient pass with a
// workgroup limit (cdsgd_plan_set_max_workgroups), which is meant to run beside other kernels, is launched without
// the bound, a compressed one with a smaller one (compressed_launch).
constexpr unsigned kLdsFor20Waves = 8192;
constexpr unsigned kLdsFor22Waves = 7168;
constexpr unsigned kLdsFor26Waves = 6144;

inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// Do [a, a + na) and [b, b + nb) share a byte?  (NULL never overlaps.)
inline bool overlap2(const void *a, size_t na, const void *b, size_t nb)
{
    if (!a || !b) return false;
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y ? y - x < na : x - y < nb;
}

// Do the byte ranges [a, a + bytes) and [b, b + bytes) share a byte?  (NULL never overlaps.)
inline bool overlap(const void *a, const void *b, size_t bytes)
{
    if (!a || !b) return false;
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y ? y - x < bytes : x - y < bytes;
}

inline unsigned long long packed_bytes_of(size_t n) { return 4ull * ((n + 15) / 16); }

// Chunks needed to cover a tensor's packed stream (which covers its elements):
// n / kChunkElems full ones, plus one for the ragged end if there is one.
inline unsigned long long chunks_of(size_t n) { return (packed_bytes_of(n) + kChunkQuads - 1) / kChunkQuads; }

inline Extent extent_of(size_t n)
{
    Extent e;
    const unsigned long long full = n / kChunkElems;
    e.full_chunks = (unsigned)full;
    e.tail_elems = (unsigned)(n - full * kChunkElems);
    e.tail_bytes = (unsigned)(packed_bytes_of(n) - full * kChunkQuads);
    e.pad_ = 0;
    return e;
}

// The same in units of `unit_quads` quads (the single-tensor kernels' pieces).
inline unsigned long long units_of(size_t n, unsigned unit_quads)
{
    return (packed_bytes_of(n) + unit_quads - 1) / unit_quads;
}

inline Extent extent_of_units(size_t n, unsigned unit_quads)
{
    Extent e;
    const unsigned long long full = n / (4ull * unit_quads);
    e.full_chunks = (unsigned)full;
    e.tail_elems = (unsigned)(n - full * 4ull * unit_quads);
    e.tail_bytes = (unsigned)(packed_bytes_of(n) - full * unit_quads);
    e.pad_ = 0;
    return e;
}

// Most chunks (or segments) a tensor or a layer list may have: a launch of one workgroup of up to
// 1024 lanes per chunk stays below 2^32 threads (1.7e10 elements).
constexpr unsigned long long kMaxGrid = 0xFFFFFFFFull / 1024;
constexpr unsigned kQuantLanes = 64;   // lanes = quads of a piece of k_quantize_pack
constexpr unsigned kUpdateLanes = 64;  // ... and of k_update
// Tensors and lists of more tiles (1024 elements each) than this are long: their streams pass the 256 MB
// memory-side cache by far, and the order in which they are read and written decides.
constexpr unsigned kLongListTiles = 28u * 1024u;
constexpr unsigned kMidListTiles = 16u * 1024u;  // where the residency of most compressed passes begins to matter

// A threshold 2^e (moderate e): every multiple m*t, |m| <= 2*CDSGD_MAX_WORKERS, is exact.
inline bool is_pow2_threshold(float t)
{
    int e = 0;
    const float m = std::frexp(t, &e);
    return m == 0.5f && e > -100 && e < 100;
}

// A threshold whose half may not be exact (the chain form's multipliers are 2, see chain_pairs).
inline bool is_tiny_threshold(float t) { return t < 0x1p-125f; }

inline bool good_threshold(float t) { return std::isfinite(t) && t > 0.0f; }

inline bool good_step_params(long step, int k, float threshold, float lr_local, float lr_global)
{
    return k >= 1 && step >= 0 && good_threshold(threshold) && std::isfinite(lr_local) && std::isfinite(lr_global);
}

inline int launch_status()
{
    return hipGetLastError() == hipSuccess ? CDSGD_OK : CDSGD_ERR_DEVICE;
}

}  // namespace

// What a pass needs to know about a layer list: device tables and a few host-side facts.
// A plan owns one (tables in memory it allocated); the entry point that allocates nothing
// builds one on the stack, its tables in the library's static device array.
struct PlanTables {
    TensorDesc *tensors = nullptr;
    ChunkRef *chunks = nullptr;
    ArenaChunk *arena_chunks = nullptr;  // the same chunks of a list in arenas, or null
    const uint8_t **rows = nullptr;     // [num_tensors][row_entries(num_workers)], null where nothing is loaded
    const void **peer_grads = nullptr;  // [num_tensors][num_workers - 1], or null: correction passes read agg_full
    int num_tensors = 0;
    int num_workers = 0;
    int self = 0;
    unsigned first_chunk = 0;           // a pass covers chunks [first_chunk, first_chunk + num_chunks) of the table
    unsigned num_chunks = 0;
    bool has_agg_full = false;
    int grad_type = kGradF32;          // element type of grad and of the bound peer gradients
    bool own_thresholds = false;       // every tensor carries its own threshold
    bool own_thresholds_pow2 = false;  // ... and all of them are powers of two
    bool own_thresholds_tiny = false;  // ... and the half of some may not be exact
    unsigned max_workgroups = 0;       // > 0: launch at most this many workgroups (they take several chunks each)
    bool peers_sparse = false;         // the peers' streams are in the sparse form (cdsgd_plan_set_peer_format)

    // Workgroups of `lanes` lanes to launch for `units` units of work (pieces of chunks): one per unit,
    // unless the plan has a limit or the launch would pass 2^32 - 1 threads (the kernels walk the units
    // with the grid's stride, so fewer workgroups than units is always correct).
    const ChunkRef *chunk_table() const { return chunks + first_chunk; }
    template <int HOW>
    auto table_for() const
    {
        if constexpr ((HOW & kArena) != 0) return (const ArenaChunk *)(arena_chunks + first_chunk);
        else return chunk_table();
    }
    bool has_arenas() const { return arena_chunks != nullptr && !own_thresholds && !peers_sparse; }

    unsigned grid_size(unsigned long long units, unsigned lanes) const
    {
        unsigned long long cap = 0xFFFFFFFFull / lanes;
        if (max_workgroups != 0 && max_workgroups < cap) cap = max_workgroups;
        return (unsigned)(units < cap ? units : cap);
    }
};

struct cdsgd_plan : PlanTables {
    void *device_block = nullptr;          // one allocation: tensors, chunks, peer pointers
    void *peer_grads_block = nullptr;      // second allocation, made by cdsgd_plan_bind_full_grads
    std::vector<TensorDesc> host_tensors;  // host copy of the descriptor table (for cdsgd_plan_set_thresholds)
    std::vector<unsigned> chunk_start;     // chunk_start[i] = first chunk of tensor i; num_tensors + 1 entries
};

struct cdsgd_trainer {
    cdsgd_plan *plan = nullptr;
    long warmup_steps = 0;
    int k = 1;
    float threshold = 0.0f, lr_local = 0.0f, lr_global = 0.0f;
    long iteration = 0;
};

namespace {

// Whether every peer's stream of checked tensors is there, is aligned and lies off this worker's buffers; false where one may
// not be (check_layer_list then says which fault comes first).  A call that makes its tables anew looks at all of them, and this is
// most of what it takes on small layers: no branches, and one comparison for each buffer, against the interval of addresses from
// which a stream of the tensor's length would reach into it.  us, cdsgd_step_fused_static on a ResNet-20-shaped list (65 tensors), the
// pointers looked at one by one here and in in_arenas / so:  N = 4 5.03 / 4.87, 8 5.65 / 5.28, 16 6.93 / 5.99, 32 9.6 / 7.7, 64 14.7 / 10.75.
bool streams_are_clear(const cdsgd_tensor *tensors, int num_tensors, const uint32_t *const *const *peers, int num_workers, int self)
{
    constexpr int kAtATime = 128, kBuffers = 4;
    uintptr_t from[kBuffers][kAtATime], span[kBuffers][kAtATime];
    for (int first = 0; first < num_tensors; first += kAtATime) {
        const int count = num_tensors - first < kAtATime ? num_tensors - first : kAtATime;
        for (int i = 0; i < count; ++i) {
            const cdsgd_tensor &t = tensors[first + i];
            const uintptr_t fb = t.n * sizeof(float), pb = (uintptr_t)packed_bytes_of(t.n);
            const void *buffer[kBuffers] = {t.w_global, t.w_local, t.residual, t.packed_self};
            for (int b = 0; b < kBuffers; ++b) {
                from[b][i] = reinterpret_cast<uintptr_t>(buffer[b]) - pb + 1u;
                span[b][i] = (b == kBuffers - 1 ? pb : fb) + pb - 1u;
            }
        }
        for (int j = 0; j < num_workers; ++j) {
            if (j == self) continue;
            if (!peers[j]) return false;
            const uint32_t *const *streams = peers[j] + first;
            uintptr_t bad = 0;
            for (int i = 0; i < count; ++i) {
                const uintptr_t p = reinterpret_cast<uintptr_t>(streams[i]);
                bad |= (p & 3u) | (uintptr_t)(p == 0);
                for (int b = 0; b < kBuffers; ++b) bad |= (uintptr_t)(p - from[b][i] < span[b][i]);
            }
            if (bad) return false;
        }
    }
    return true;
}

// Host-side checks of a layer list and its peers (no HIP call): what cdsgd_plan_create_typed
// and cdsgd_step_fused_static share.  Returns the number of chunks and whether every tensor
// has an agg_full buffer.
int check_layer_list(const cdsgd_tensor *tensors, int num_tensors, const uint32_t *const *const *peers,
                     int num_workers, int self, int grad_dtype, unsigned long long *total_chunks_out,
                     bool *all_agg_out)
{
    if (!tensors) return CDSGD_ERR_NULL;
    if (grad_dtype != CDSGD_GRAD_F32 && grad_dtype != CDSGD_GRAD_BF16 && grad_dtype != CDSGD_GRAD_F16)
        return CDSGD_ERR_PARAM;
    const size_t grad_elem = grad_dtype == CDSGD_GRAD_F32 ? 4 : 2;
    if (num_tensors < 1) return CDSGD_ERR_SIZE;
    if (num_workers < 1 || num_workers > CDSGD_MAX_WORKERS || self < 0 || self >= num_workers)
        return CDSGD_ERR_WORKERS;
    if (num_workers > 1 && !peers) return CDSGD_ERR_NULL;
    unsigned long long total_chunks = 0;
    bool all_agg = true;
    for (int i = 0; i < num_tensors; ++i) {
        const cdsgd_tensor &t = tensors[i];
        if (!t.w_global || !t.w_local || !t.residual || !t.grad || !t.packed_self) return CDSGD_ERR_NULL;
        if (t.n == 0 || chunks_of(t.n) > kMaxGrid) return CDSGD_ERR_SIZE;
        if (!aligned(t.w_global, 16) || !aligned(t.w_local, 16) || !aligned(t.residual, 16) ||
            !aligned(t.grad, 16) || !aligned(t.agg_full, 16) || !aligned(t.packed_self, 4))
            return CDSGD_ERR_ALIGN;
        const size_t fb = t.n * sizeof(float), gb = t.n * grad_elem, pb = (size_t)packed_bytes_of(t.n);
        if (overlap(t.w_global, t.w_local, fb) || overlap(t.w_global, t.residual, fb) ||
            overlap(t.w_local, t.residual, fb) || overlap(t.agg_full, t.w_global, fb) ||
            overlap(t.agg_full, t.w_local, fb) || overlap2(t.grad, gb, t.residual, fb) ||
            overlap2(t.grad, gb, t.w_global, fb) || overlap2(t.grad, gb, t.w_local, fb) ||
            overlap2(t.packed_self, pb, t.w_global, fb) || overlap2(t.packed_self, pb, t.w_local, fb) ||
            overlap2(t.packed_self, pb, t.residual, fb) || overlap2(t.packed_self, pb, t.grad, gb) ||
            overlap2(t.packed_self, pb, t.agg_full, fb))
            return CDSGD_ERR_ALIAS;
        all_agg = all_agg && t.agg_full != nullptr;
        total_chunks += chunks_of(t.n);
        if (total_chunks > kMaxGrid) return CDSGD_ERR_SIZE;
    }
    *total_chunks_out = total_chunks;
    *all_agg_out = all_agg;
    if (streams_are_clear(tensors, num_tensors, peers, num_workers, self)) return CDSGD_OK;
    for (int j = 0; j < num_workers; ++j) {
        if (j == self) continue;
        if (!peers[j]) return CDSGD_ERR_NULL;
        for (int i = 0; i < num_tensors; ++i) {
            if (!peers[j][i]) return CDSGD_ERR_NULL;
            if (!aligned(peers[j][i], 4)) return CDSGD_ERR_ALIGN;
            // a peer's stream is read while this tensor's outputs are written
            const cdsgd_tensor &t = tensors[i];
            const size_t fb = t.n * sizeof(float), pb = (size_t)packed_bytes_of(t.n);
            if (overlap2(peers[j][i], pb, t.w_global, fb) || overlap2(peers[j][i], pb, t.w_local, fb) ||
                overlap2(peers[j][i], pb, t.residual, fb) || overlap2(peers[j][i], pb, t.packed_self, pb))
                return CDSGD_ERR_ALIAS;
        }
    }
    return CDSGD_OK;
}

TensorDesc make_desc(const cdsgd_tensor &t)
{
    TensorDesc d;
    d.w_global = t.w_global;
    d.w_local = t.w_local;
    d.residual = t.residual;
    d.grad = t.grad;
    d.packed_self = reinterpret_cast<uint8_t *>(t.packed_self);
    d.agg_full = t.agg_full;
    d.ext = extent_of(t.n);
    d.threshold = 0.0f;
    d.pad_ = 0;
    return d;
}

// The offset, in 16 elements, of tensor i's buffers from tensor 0's if every one of its own is that far (agg_full
// everywhere or nowhere) and the arenas' packed streams are below 4 GiB, -1 if not.
long long arena_offset16(const cdsgd_tensor *tensors, int i, unsigned grad_bytes)
{
    const cdsgd_tensor &z = tensors[0], &t = tensors[i];
    const auto diff = [](const void *a, const void *b) {
        return (long long)(reinterpret_cast<uintptr_t>(a) - reinterpret_cast<uintptr_t>(b));
    };
    const long long bytes = diff(t.w_global, z.w_global);
    if (bytes < 0 || bytes % 64 != 0 || bytes / 64 > 0x3FFFFFFFll) return -1;
    const long long off = bytes / 64;
    if ((unsigned long long)off * 4ull + packed_bytes_of(t.n) > 0xFFFFFFFFull) return -1;
    if (diff(t.w_local, z.w_local) != bytes || diff(t.residual, z.residual) != bytes ||
        diff(t.grad, z.grad) != off * 16 * (long long)grad_bytes || diff(t.packed_self, z.packed_self) != off * 4)
        return -1;
    if ((t.agg_full == nullptr) != (z.agg_full == nullptr) || (t.agg_full && diff(t.agg_full, z.agg_full) != bytes))
        return -1;
    return off;
}

// ... of all tensors of a list into `offsets`, or false.
bool in_arenas(const cdsgd_tensor *tensors, int num_tensors, const uint32_t *const *const *peers, int num_workers, int self,
               unsigned grad_bytes, unsigned *offsets)
{
    offsets[0] = 0u;
    for (int i = 1; i < num_tensors; ++i) {
        const long long off = arena_offset16(tensors, i, grad_bytes);
        if (off < 0) return false;
        offsets[i] = (unsigned)off;
    }
    for (int j = 0; j < num_workers; ++j) {  // worker by worker, as the pointers lie
        if (j == self) continue;
        uintptr_t other = 0;
        const uintptr_t zero = reinterpret_cast<uintptr_t>(peers[j][0]);
        for (int i = 1; i < num_tensors; ++i)
            other |= (reinterpret_cast<uintptr_t>(peers[j][i]) - zero) ^ ((uintptr_t)offsets[i] * 4u);
        if (other) return false;
    }
    return true;
}

// LDS bound of a pass that sums the workers' gradients in the kernel.  Measured, time of the pass with 26 waves per
// compute unit over its time with 0 (32 waves) / 6 / 7 / 8 KiB (26, 22 and 20 waves):
//   32-bit   VGG-16-shaped, N = 4 / 8 / 16   0.99 0.99 0.97 / 1.00 1.00 1.00 / 1.02 1.02 1.02 / 1.04 1.05 1.00
//            25 M elements, N = 8 / 16       0.99 0.99 / 1.00 1.01 / 1.01 1.02 / 1.00 1.00
//            4 M elements, N = 8 / 16        1.01 1.01 / 1.01 1.01 / 0.95 0.94 / 0.97 0.98
//   16-bit   VGG-16-shaped, N = 8 / 16       0.99 1.05 / 1.00 1.07 / 1.01 1.08 / 1.02 1.07
//   (pairs)  25 M elements, N = 8 / 16       1.04 1.08 / 1.04 1.08 / 1.03 1.07 / 1.02 1.05;  N = 2 0.98 / 1.00 / 1.00 / 1.00
//            4 M elements, N = 8             1.13 / 1.10 / 1.02 / 1.02
unsigned lds_of_kernel_sum(unsigned num_chunks, int num_workers, int grad_type)
{
    const unsigned tiles = num_chunks * kTilesPerChunk;
    const bool short_list = tiles <= 6u * 1024u, long_list = tiles > kLongListTiles;
    if (grad_type != kGradF32) return short_list ? 0u : (long_list ? kLdsFor22Waves : kLdsFor26Waves);
    if (short_list) return kLdsFor26Waves;
    return long_list && num_workers <= 8 ? kLdsFor20Waves : kLdsFor22Waves;
}

// Whether a correction pass (gradients of any type) writes its results through, the global weights staying in the memory-side
// cache and the local ones not, instead of storing both non-temporally.  A program that corrects every k steps finds none of a
// list's buffers in that cache, a small one that does little else may find all, so the line lies where neither loses.
// Time over that of non-temporal stores: three sets of buffers in turn (up to some million elements they fit the cache) /
// 600 MB of sets / 1500 MB of sets:
//   sum, N = 2, 32-bit   0.5 M .99 / 1.02 / 1.00, 1 M .91 / 1.00 / 1.02, 3 M .99 / 1.00 / 1.01, 6 M .98 / .96 / 1.02, 14 M .96 / .96 / .97
//   sum, N = 2, bf16     0.5 M 1.00 / 1.01 / 1.00, 1 M .99 / 1.00 / 1.04, 1.9 M .76 / .99 / 1.10, 3 M .99 - 1.03 / 1.03 / .99 - 1.09, 6 M 1.01 / .98 / 1.01,
//                        14 M .96 / .96 / 1.02
//   sum, N = 4, 32-bit   0.5 M .98 / 1.10 / 1.07, 1 M 1.03 / 1.07 / 1.05, 3 M .99 / .99 / .98, 6 M .95 / .95 / .94, 14 M .93 / .94 / .93
//   sum, N = 4, bf16     0.5 M 1.00 / 1.07 / 1.07, 1 M .89 / 1.10 / 1.11, 3 M .97 / 1.03 / 1.08, 6 M 1.00 / .98 / 1.05, 14 M .94 / .95 / .97
//   agg_full             0.5 M .99 / .99 / 1.02, 1 M .81 / 1.03 / 1.04, 4 M 1.01 / .97 / 1.03, 8 M .97 / .95 / .98, 13 M .96 / .96 / .99
//   sum, N = 8 / 16      0.3 to 1.9 M, 32-bit .94 to 1.01 / .99 to 1.15 / 1.04 to 1.14;  bf16 .92 to 1.00 / 1.10 to 1.23 / 1.10 to 1.20
//   sum, lists that fit no cache   75 M 1.00;  100 M N = 5 .99 - 1.01, 8 .99 - 1.01, 16 .99;  130 M .98 - 1.00;  VGG-16 N = 5 .99 - 1.01, 8 .97 - .99,
//                        12 .98 - 1.02, 16 .95 - 1.00
// (both staying: 14 M 1.03, and 1 to 2 M 2 to 14 % slower than so where the sets do not fit)
bool keeps_results(unsigned num_chunks, int num_workers, bool sum)
{
    const unsigned tiles = num_chunks * kTilesPerChunk;
    if (sum && num_workers > 4) return tiles > 72u * 1024u;
    return tiles > (sum && num_workers > 2 ? 4u * 1024u : 768u) && tiles <= 14u * 1024u;
}

// Whether a pass that sums the workers' gradients asks for several workers' at once (kTogether): on short lists, which have
// too few waves to keep the memory busy with one load (16-bit gradients: two) in flight each.  Time over that in order, three
// sets of buffers in turn (N = 16 in us):
//   32-bit   N = 6   0.1 M .98, 0.5 M .80, 0.7 M .93, 1 M .95, 1.5 M 1.00, 3 M 1.03      N = 8   .92, .72, .88, .97, 1.04, 1.05
//            N = 16  0.1 M 7.6 / 4.0, 0.25 M 13.0 / 7.5, 0.5 M 10.5 / 7.1, 0.7 M 11.6 / 9.6, 1 M 13.7 / 13.1, 1.5 M 18.2 / 19.5
//   16-bit   N = 6   0.5 M .99, 0.7 M 1.00, 1 M 1.04 (600 MB of sets .97), 2 M 1.07       N = 8   .94, .92, .96, 1.03
//            N = 16  0.25 M 6.3 / 4.6, 0.5 M 7.0 / 5.3, 0.7 M 7.9 / 6.4, 1 M 8.9 / 8.3, 1.5 M 11.3 / 11.5
// and on either side of the lines
//   32-bit   N = 5   0.25 M .79, 0.5 M .81, 0.65 M .92, 0.75 M 1.01, 1 M 1.00      N = 7   0.25 M .66, 0.5 M .78, 0.75 M .93, 1 M .96, 1.2 M 1.03
//   16-bit   N = 5   0.25 M 1.04, 0.5 M 1.06, 0.75 M 1.06, 1 M 1.11, 2 M 1.01      N = 7   0.25 M .93, 0.5 M .83, 0.75 M .90, 1 M .91, 2 M 1.03
// (Up to 4 workers nothing is gained and 1 M in 16 bits loses 11 %; 4 at once gain less up to 0.5 M, 16 at once are slower
// from 0.7 M on.  Above, the order of the streams decides: 8 M, N = 16 92 / 107.)
bool sums_together(unsigned num_chunks, int num_workers, int grad_type)
{
    return num_workers > (grad_type == kGradF32 ? 4 : 5) && num_chunks * kTilesPerChunk <= (num_workers > 6 ? 1024u : 768u);
}

// Launch one full-gradient pass (see k_fused_full) for a plan.
int launch_full_pass(const PlanTables *plan, int local_mode, float lr_local, float lr_global, void *hip_stream)
{
    const bool sum = plan->peer_grads != nullptr || plan->num_workers == 1;
    if (!sum && !plan->has_agg_full) return CDSGD_ERR_NULL;
    const float scale = lr_global / (float)plan->num_workers;
    hipStream_t s = (hipStream_t)hip_stream;
    const unsigned long long num_pieces = (unsigned long long)plan->num_chunks * kPiecesPerChunk;
    const dim3 grid(plan->grid_size(num_pieces, kFullBlock)), block(kFullBlock);
    const int np = plan->num_workers - 1;
    // a pass with a workgroup limit is meant to share the GPU with other kernels: it leaves the LDS to them
    const unsigned lds_plain = plan->max_workgroups ? 0u : kLdsFor20Waves;
    const unsigned lds_sum = plan->max_workgroups ? 0u : lds_of_kernel_sum(plan->num_chunks, plan->num_workers, plan->grad_type);
#define CDSGD_LAUNCH_FULL_T(SUM, LOCAL, GT, STORE, IN_FLIGHT)                                                  \
    hipLaunchKernelGGL((k_fused_full<SUM, LOCAL, GT, STORE, IN_FLIGHT>), grid, block, (SUM ? lds_sum : lds_plain), s,   \
                       plan->tensors, plan->chunk_table(),                                                      \
                       num_pieces, plan->peer_grads, np, plan->self, lr_local, scale)
#define CDSGD_LAUNCH_FULL(SUM, LOCAL, STORE, IN_FLIGHT)                                                        \
    do {                                                                                                       \
        if (plan->grad_type == kGradBF16) CDSGD_LAUNCH_FULL_T(SUM, LOCAL, kGradBF16, STORE, IN_FLIGHT);        \
        else if (plan->grad_type == kGradF16) CDSGD_LAUNCH_FULL_T(SUM, LOCAL, kGradF16, STORE, IN_FLIGHT);     \
        else CDSGD_LAUNCH_FULL_T(SUM, LOCAL, kGradF32, STORE, IN_FLIGHT);                                      \
    } while (0)
    const bool keep = plan->max_workgroups == 0 && keeps_results(plan->num_chunks, plan->num_workers, sum);
    if (sum && sums_together(plan->num_chunks, plan->num_workers, plan->grad_type)) {
        if (local_mode == kLocalNone) CDSGD_LAUNCH_FULL(true, kLocalNone, kStream, kTogether);
        else if (local_mode == kLocalCopy) CDSGD_LAUNCH_FULL(true, kLocalCopy, kStream, kTogether);
        else CDSGD_LAUNCH_FULL(true, kLocalRule, kStream, kTogether);
    } else if (sum) {
        if (local_mode == kLocalNone) CDSGD_LAUNCH_FULL(true, kLocalNone, kStream, kInOrder);
        else if (local_mode == kLocalCopy) CDSGD_LAUNCH_FULL(true, kLocalCopy, kStream, kInOrder);
        else if (keep) CDSGD_LAUNCH_FULL(true, kLocalRule, kThrough, kInOrder);
        else CDSGD_LAUNCH_FULL(true, kLocalRule, kStream, kInOrder);
    } else {
        if (local_mode == kLocalNone) CDSGD_LAUNCH_FULL(false, kLocalNone, kStream, kInOrder);
        else if (local_mode == kLocalCopy) CDSGD_LAUNCH_FULL(false, kLocalCopy, kStream, kInOrder);
        else if (keep) CDSGD_LAUNCH_FULL(false, kLocalRule, kThrough, kInOrder);
        else CDSGD_LAUNCH_FULL(false, kLocalRule, kStream, kInOrder);
    }
#undef CDSGD_LAUNCH_FULL
#undef CDSGD_LAUNCH_FULL_T
    return launch_status();
}

// Whether decode-and-sum and the global rule behind it store non-temporally: few workers' sums of a few million elements,
// which pass from call to call through the dies' own caches.  (Neither call knows whether the streams of the other are
// packed or sparse, so the line lies where nothing loses against non-temporal stores throughout.)  Both calls, stored so /
// written through and staying, us, packed streams unless said:
//   N = 2    1.6 M 8.2 / 8.5, 2 M 8.4 / 9.9, 4 M 12.0 / 12.6, 5 M 14.7 / 14.3      N = 4 (sparse)  4 M 12.4 / 12.8, 5 M 15.4 / 14.5
//   N = 8    1.6 M 8.1 / 8.6, 2.2 M 8.8 / 9.3, 2.7 M 10.0 / 10.1, 3.5 M 12.7 / 12.1
//   N = 12   1.6 M 8.1 / 8.7, 2.2 M 9.2 / 8.7, 2.7 M 10.6 / 10.1
//   N = 16, sparse, one code in 256   1.6 M 8.3 / 9.3, 2.2 M 9.6 / 10.8, 3 M 11.5 / 11.8, 3.5 M 13.4 / 12.9; one in 16
//            1.6 M 8.5 / 8.7, 2.2 M 10.5 / 9.9
//   N = 32, sparse, one code in 256   1.6 M 9.4 / 9.5, 2.2 M 11.0 / 10.9;  N = 64 1.6 M 12.2 / 12.1;  0.1 M, N = 4 4.7 / 4.4
inline bool drains_results(size_t n, int num_workers)
{
    const size_t most = num_workers <= kUpTo4 ? 4500000u : (num_workers <= kUpTo16 ? 3200000u : (num_workers <= kUpTo32 ? 1750000u : 0u));
    return n > 1250000u && n <= most;
}

// Whether the weights that the global rule writes stay in the memory-side cache for the next one: not where they push out
// streams that a later decode-and-sum would find there, and not where few programs come back before they are pushed out
// themselves.  Decode-and-sum and update, time over that of non-temporal stores in both, weights staying, then not staying:
//   three / four sets of buffers in turn
//     N = 33   5 M .92 / .96, .94 / .94;  6 M .95 / 1.01, .95 / .94;  7 M .99 / 1.01, .95 / .96
//     N = 48   4 M .94 / 1.04, .96 / .98;  5 M 1.00 / 1.03, .96 / .98;  6 M 1.01 / 1.05, .97 / .94;  7 M 1.04 / 1.05, .97 / .94
//     N = 64   3 M .96 / .99, .97 / .97;  4 M 1.00 / 1.04, .98 / .98;  5 M 1.04 / 1.01, .99 / .90;  6 M 1.08 / 1.01, .96 / .94
//     N = 64, sparse, one code in 16   4 M .97 / 1.13, .96 / .99;  6 M 1.12 / 1.02, .99 / .95
//   (With two sets, which fit, staying is 2 % faster throughout.)
//   three sets / 1500 MB of sets
//     N = 2    5 M .97 / .93, 1.05 / .94;  6.5 M .92 / .95, 1.00 / .95      N = 4    5 M .95 / .97, 1.01 / .94;  6.5 M .92 / 1.00, .97 / .94
//     N = 8    4 M .93 / 1.00, .97 / .95;  5 M .92 / 1.00, .95 / .96;  6.5 M .91 / 1.03, .96 / .95;  sparse 6 M .93 / 1.07, .96 / .93
//     N = 16   5 M .92 / .98, .95 / .95;  sparse 6 M .93 / 1.02, .95 / .94       N = 24   6.5 M .91 / .95, .95 / .94
inline bool weights_stay(size_t n, int num_workers)
{
    return n <= (num_workers <= kUpTo4 ? kSmallElems : (size_t)5000000u) &&
           (unsigned long long)num_workers * packed_bytes_of(n) <= 48000000ull;
}

// a4 for one tensor on checked arguments.
//
// Tiles of a group: 4 up to 16 workers; above that the loads of a wave are enough with one tile of packed streams
// (N = 32, 2^27 elements, t = 0.5: 0.268 ms, 0.277 with 2 tiles) and want two of sparse ones (N = 24, one code in 256:
// 0.277 ms with one, 0.230 with 2), except in the chain form above 32 workers, where a tile's rows and sums take 20 KiB
// (N = 64: 0.65 ms, 0.70 with 2).
// LDS that a group asks for in all, which bounds the groups resident (kLdsFor20Waves): with more than 4 packed streams
// the mix of reads and writes is served better with 5 groups in the count form (N = 8, 2^27 elements: 133 us with all
// groups, 127 with 5) and 6 in the chain form (N = 9: 140 with all, 136 with 6, 144 with 5), above 8 workers from 16 M
// elements on (N = 16: 9 M 17.8 us with all, 18.4 with 6; 25 M 40.0 and 39.5); 4 streams and fewer write mostly and
// lose with any bound (N = 2: 96 us, 113 with 5); sparse streams gain in the count form (N = 12, one code in 4: 173 us,
// 169 with 6) and lose in the chain form; above 32 workers the count form gains from 16 M elements on (N = 64, 60 M:
// decode-and-sum and update 288 us with all, 283 with 5).
// Packed streams are read non-temporally when they are more than the caches between the workers' data and the compute
// units hold on to: above 56 MB, and above 100 MB with more than 16 workers, whose sums write little (decode-and-sum and
// update, default policy / non-temporal, us: N = 4, 32 M 77.3 / 79.0, 60 M 145.5 / 143.4;  N = 8, 25 M 66.3 / 67.7, 32 M
// 86.4 / 84.1;  N = 9, 20 M 53.2 / 54.3, 25 M 69.5 / 68.2;  N = 12, 10 M 30.0 / 31.8, 60 M 167 / 161;  N = 24, 5 M 18.4 /
// 20.0, 14 M the same;  N = 32, 10 M 40.2 / 40.6, 16 M 66.6 / 64.0;  N = 48, 7 M 31.6 / 33.0, 10 M 46.0 / 44.2;  N = 64,
// 7 M the same, 14 M 76.3 / 72.0).
template <bool SPARSE>
int launch_decode_sum(const uint32_t *const *streams, int num_workers, float *agg, size_t n, float threshold, void *hip_stream)
{
    StreamTable tab;
    std::memset(&tab, 0, sizeof(tab));
    for (int j = 0; j < num_workers; ++j) tab.p[j] = reinterpret_cast<const uint8_t *>(streams[j]);
    const unsigned tiles = (unsigned)units_of(n, kTileQuads);
    const Extent ext = extent_of(n);
    const int drain = drains_results(n, num_workers) ? 1 : 0;
    const int xcd = SPARSE || tiles > kLongListTiles ? 1 : 0;
    const bool nt = !SPARSE && (unsigned long long)num_workers * packed_bytes_of(n) > (num_workers > kUpTo16 ? 100000000ull : 56000000ull);
    hipStream_t s = (hipStream_t)hip_stream;
#define CDSGD_LAUNCH_DECODE(SZ, FORM, TILES, LDS)                                                              \
    do {                                                                                                       \
        const unsigned groups = (tiles + TILES - 1u) / TILES, used = kTileLds<SZ, FORM, 4, SPARSE, false> * TILES, want = LDS; \
        const unsigned more = want > used ? want - used : 0u;                                                   \
        if (!SPARSE && nt)                                                                                      \
            hipLaunchKernelGGL((k_decode_sum<SZ, FORM, SPARSE, TILES, !SPARSE>), dim3(groups), dim3(kTileQuads), \
                               more, s, agg, ext, num_workers, groups, xcd, drain, threshold, tab);                    \
        else                                                                                                    \
            hipLaunchKernelGGL((k_decode_sum<SZ, FORM, SPARSE, TILES, false>), dim3(groups), dim3(kTileQuads),  \
                               more, s, agg, ext, num_workers, groups, xcd, drain, threshold, tab);                    \
    } while (0)
    const bool count = is_pow2_threshold(threshold);
    constexpr unsigned kLdsCount = SPARSE ? 24576u : 32768u, kLdsChain = SPARSE ? 0u : 24576u;
    constexpr int kTilesMany = SPARSE ? 2 : 1;
    // (Thresholds whose half may not be exact have the shapes of the other chains; 25 M elements, packed, us, with the kernel
    // for any number of workers / so: N = 2 43.7 / 21.1, 8 41.2 / 28.8, 16 44.0 / 38.0, 17 46.5 / 42.1, 24 51.3 / 48.2,
    // 32 59.4 / 58.3;  sparse N = 16 55.9 / 41.5, 24 68.6 / 57.1.)
    const bool tiny = !count && is_tiny_threshold(threshold);
#define CDSGD_LAUNCH_DECODE_CHAIN(SZ, TILES, LDS)                                                              \
    do {                                                                                                       \
        if (tiny) CDSGD_LAUNCH_DECODE(SZ, kChainTiny, TILES, LDS);                                             \
        else CDSGD_LAUNCH_DECODE(SZ, kChain, TILES, LDS);                                                      \
    } while (0)
    if (num_workers <= kUpTo4) {
        if (count) CDSGD_LAUNCH_DECODE(kUpTo4, kCount, 4, 0u);
        else CDSGD_LAUNCH_DECODE_CHAIN(kUpTo4, 4, 0u);
    } else if (num_workers <= kUpTo8) {
        if (count) CDSGD_LAUNCH_DECODE(kUpTo8, kCount, 4, kLdsCount);
        else CDSGD_LAUNCH_DECODE_CHAIN(kUpTo8, 4, kLdsChain);
    } else if (num_workers <= kUpTo16) {
        if (count) CDSGD_LAUNCH_DECODE(kUpTo16, kCount, 4, kLdsCount);
        else CDSGD_LAUNCH_DECODE_CHAIN(kUpTo16, 4, (tiles > kMidListTiles ? kLdsChain : 0u));
    } else if (num_workers <= kUpTo32) {
        if (count) CDSGD_LAUNCH_DECODE(kUpTo32, kCount, kTilesMany, 0u);
        else CDSGD_LAUNCH_DECODE_CHAIN(kUpTo32, kTilesMany, 0u);
    } else {
        if (count) CDSGD_LAUNCH_DECODE(kAnyWorkers, kCount, kTilesMany, (!SPARSE && tiles > kMidListTiles ? kLdsCount : 0u));
        else CDSGD_LAUNCH_DECODE_CHAIN(kAnyWorkers, 1, 0u);
    }
#undef CDSGD_LAUNCH_DECODE_CHAIN
#undef CDSGD_LAUNCH_DECODE
    return launch_status();
}

}  // namespace

#ifndef CDSGD_BUILD_ID_HEX
#define CDSGD_BUILD_ID_HEX "0000000000000000"
#endif

extern "C" {

size_t cdsgd_packed_words(size_t n) { return (n + 15) / 16; }

// The marker in front makes the identity findable in the file without loading it.
const char *cdsgd_build_id(void)
{
    static const char id[] = "CDSGD_BUILD_ID=" CDSGD_BUILD_ID_HEX;
    return id + 15;
}

const char *cdsgd_status_string(int status)
{
    switch (status) {
    case CDSGD_OK: return "ok";
    case CDSGD_ERR_NULL: return "a required pointer is NULL";
    case CDSGD_ERR_SIZE:
        return "bad size (zero elements, no tensors, too large for one launch, or beyond the limits of "
               "cdsgd_step_fused_static's tables)";
    case CDSGD_ERR_PARAM: return "bad parameter (threshold, k, step or learning rate)";
    case CDSGD_ERR_ALIGN: return "pointer not aligned (fp32 buffers 16 bytes, packed buffers 4 bytes)";
    case CDSGD_ERR_WORKERS: return "bad worker count or worker index";
    case CDSGD_ERR_DEVICE: return "a HIP call failed";
    case CDSGD_ERR_ALIAS: return "buffers that must be distinct overlap";
    default: return "unknown status";
    }
}

int cdsgd_quantize_pack(const float *grad, float *residual, uint32_t *packed, size_t n, float threshold,
                        void *hip_stream)
{
    if (!grad || !residual || !packed) return CDSGD_ERR_NULL;
    if (n == 0 || units_of(n, kQuantLanes) > 0xFFFFFFFFull / kQuantLanes) return CDSGD_ERR_SIZE;
    if (!good_threshold(threshold)) return CDSGD_ERR_PARAM;
    if (!aligned(grad, 16) || !aligned(residual, 16) || !aligned(packed, 4)) return CDSGD_ERR_ALIGN;
    if (overlap(grad, residual, n * sizeof(float)) ||
        overlap2(packed, (size_t)packed_bytes_of(n), grad, n * sizeof(float)) ||
        overlap2(packed, (size_t)packed_bytes_of(n), residual, n * sizeof(float)))
        return CDSGD_ERR_ALIAS;
    const dim3 grid((unsigned)units_of(n, kQuantLanes)), block(kQuantLanes);
    const Extent pieces = extent_of_units(n, kQuantLanes);
    hipStream_t s = (hipStream_t)hip_stream;
    uint8_t *codes = reinterpret_cast<uint8_t *>(packed);
#define CDSGD_LAUNCH_QUANT(LEN, LDS)                                                                           \
    hipLaunchKernelGGL((k_quantize_pack<kQuantLanes, LEN>), grid, block, LDS, s, grad, residual, codes, pieces, threshold)
    if (n <= kSmallElems) CDSGD_LAUNCH_QUANT(kSmallTensor, 0);
    else if (n <= kKeepElems) CDSGD_LAUNCH_QUANT(kMidTensor, kLdsFor26Waves);
    else CDSGD_LAUNCH_QUANT(kLargeTensor, kLdsFor20Waves);
#undef CDSGD_LAUNCH_QUANT
    return launch_status();
}

int cdsgd_decode_sum(const uint32_t *const *packed, int num_workers, float *agg, size_t n, float threshold,
                     void *hip_stream)
{
    if (!packed || !agg) return CDSGD_ERR_NULL;
    if (n == 0 || chunks_of(n) > kMaxGrid) return CDSGD_ERR_SIZE;
    if (!good_threshold(threshold)) return CDSGD_ERR_PARAM;
    if (num_workers < 1 || num_workers > CDSGD_MAX_WORKERS) return CDSGD_ERR_WORKERS;
    for (int j = 0; j < num_workers; ++j)
        if (!packed[j]) return CDSGD_ERR_NULL;
    if (!aligned(agg, 16)) return CDSGD_ERR_ALIGN;
    for (int j = 0; j < num_workers; ++j)
        if (!aligned(packed[j], 4)) return CDSGD_ERR_ALIGN;
    for (int j = 0; j < num_workers; ++j)
        if (overlap2(packed[j], (size_t)packed_bytes_of(n), agg, n * sizeof(float))) return CDSGD_ERR_ALIAS;
    return launch_decode_sum<false>(packed, num_workers, agg, n, threshold, hip_stream);
}

int cdsgd_update(float *w_global, float *w_local, const float *grad_local, const float *agg, size_t n,
                 float lr_local, float lr_global, int num_workers, void *hip_stream)
{
    const bool local = w_local != nullptr || grad_local != nullptr;
    const bool global = agg != nullptr;
    if (!w_global) return CDSGD_ERR_NULL;
    if (local && (!w_local || !grad_local)) return CDSGD_ERR_NULL;
    if (!local && !global) return CDSGD_ERR_NULL;
    if (n == 0 || units_of(n, kUpdateLanes) > 0xFFFFFFFFull / kUpdateLanes) return CDSGD_ERR_SIZE;
    if (!std::isfinite(lr_local) || !std::isfinite(lr_global)) return CDSGD_ERR_PARAM;
    if (num_workers < 1 || num_workers > CDSGD_MAX_WORKERS) return CDSGD_ERR_WORKERS;
    if (!aligned(w_global, 16) || !aligned(w_local, 16) || !aligned(grad_local, 16) || !aligned(agg, 16))
        return CDSGD_ERR_ALIGN;
    if (overlap(w_global, w_local, n * sizeof(float)) || overlap(w_local, grad_local, n * sizeof(float)) ||
        overlap(w_local, agg, n * sizeof(float)) || overlap(w_global, grad_local, n * sizeof(float)) ||
        overlap(w_global, agg, n * sizeof(float)))
        return CDSGD_ERR_ALIAS;
    const float scale = lr_global / (float)num_workers;
    hipStream_t s = (hipStream_t)hip_stream;
    const dim3 grid((unsigned)units_of(n, kUpdateLanes)), block(kUpdateLanes);
    const Extent pieces = extent_of_units(n, kUpdateLanes);
#define CDSGD_LAUNCH_UPDATE(LOCAL, GLOBAL, LEN, LDS)                                                           \
    hipLaunchKernelGGL((k_update<LOCAL, GLOBAL, LEN>), grid, block, LDS, s, w_global, w_local, grad_local, agg, \
                       pieces, lr_local, scale)
    const bool small = n <= kSmallElems, mid = n <= kKeepElems;
    if (local && global) {
        if (small) CDSGD_LAUNCH_UPDATE(true, true, kSmallTensor, 0);
        else if (mid) CDSGD_LAUNCH_UPDATE(true, true, kMidTensor, kLdsFor20Waves);
        else CDSGD_LAUNCH_UPDATE(true, true, kLargeTensor, kLdsFor20Waves);
    } else if (local) {
        if (small) CDSGD_LAUNCH_UPDATE(true, false, kSmallTensor, 0);
        else if (mid) CDSGD_LAUNCH_UPDATE(true, false, kMidTensor, kLdsFor26Waves);
        else CDSGD_LAUNCH_UPDATE(true, false, kLargeTensor, kLdsFor20Waves);
    } else {
        if (drains_results(n, num_workers)) CDSGD_LAUNCH_UPDATE(false, true, kDrainTensor, 0);
        else if (weights_stay(n, num_workers)) CDSGD_LAUNCH_UPDATE(false, true, kSmallTensor, 0);
        else CDSGD_LAUNCH_UPDATE(false, true, kMidTensor, 0);
    }
#undef CDSGD_LAUNCH_UPDATE
    return launch_status();
}

int cdsgd_plan_create(const cdsgd_tensor *tensors, int num_tensors, const uint32_t *const *const *peers,
                      int num_workers, int self, cdsgd_plan **out)
{
    return cdsgd_plan_create_typed(tensors, num_tensors, peers, num_workers, self, CDSGD_GRAD_F32, out);
}

int cdsgd_plan_create_typed(const cdsgd_tensor *tensors, int num_tensors, const uint32_t *const *const *peers,
                            int num_workers, int self, int grad_dtype, cdsgd_plan **out)
try {
    if (!out) return CDSGD_ERR_NULL;
    *out = nullptr;
    unsigned long long total_chunks = 0;
    bool all_agg = true;
    const int rc = check_layer_list(tensors, num_tensors, peers, num_workers, self, grad_dtype, &total_chunks, &all_agg);
    if (rc != CDSGD_OK) return rc;
    const unsigned row = row_entries(num_workers);
    const unsigned grad_bytes = grad_dtype == CDSGD_GRAD_F32 ? 4u : 2u;
    std::vector<unsigned> offsets((size_t)num_tensors);
    const bool arenas = in_arenas(tensors, num_tensors, peers, num_workers, self, grad_bytes, offsets.data());

    // host image of the device block
    const size_t bytes_t = sizeof(TensorDesc) * (size_t)num_tensors;
    const size_t bytes_c = sizeof(ChunkRef) * (size_t)total_chunks;
    // (a batch of pointers past the last row: a kernel for any number of workers reads a short row that far)
    const size_t bytes_p = sizeof(const uint8_t *) * ((size_t)num_tensors * row + CDSGD_MAX_WORKERS);
    const size_t off_c = (bytes_t + 255) & ~(size_t)255;
    const size_t off_p = (off_c + bytes_c + 255) & ~(size_t)255;
    const size_t off_a = (off_p + bytes_p + 255) & ~(size_t)255;
    const size_t total = off_a + (arenas ? sizeof(ArenaChunk) * (size_t)total_chunks : 0);
    std::vector<unsigned char> image(total, 0);
    TensorDesc *ht = reinterpret_cast<TensorDesc *>(image.data());
    ChunkRef *hc = reinterpret_cast<ChunkRef *>(image.data() + off_c);
    const uint8_t **hp = reinterpret_cast<const uint8_t **>(image.data() + off_p);
    ArenaChunk *ha = reinterpret_cast<ArenaChunk *>(image.data() + off_a);
    size_t ci = 0;
    std::vector<unsigned> chunk_start((size_t)num_tensors + 1, 0u);
    for (int i = 0; i < num_tensors; ++i) {
        const cdsgd_tensor &t = tensors[i];
        ht[i] = make_desc(t);
        const unsigned nc = (unsigned)chunks_of(t.n);
        chunk_start[(size_t)i + 1] = chunk_start[(size_t)i] + nc;
        for (unsigned c = 0; c < nc; ++c) {
            hc[ci].tensor = (unsigned)i;
            hc[ci].chunk = c;
            if (arenas) {
                const size_t left = t.n - (size_t)c * kChunkElems;
                ha[ci].off16 = offsets[(size_t)i] + c * (kChunkElems / 16u);
                ha[ci].elems = (unsigned)(left < kChunkElems ? left : kChunkElems);
            }
            ++ci;
        }
        for (int j = 0; j < num_workers; ++j)
            if (j != self) hp[(size_t)i * row + (size_t)j] = reinterpret_cast<const uint8_t *>(peers[j][i]);
    }

    std::unique_ptr<cdsgd_plan, int (*)(cdsgd_plan *)> plan(new cdsgd_plan, cdsgd_plan_destroy);
    plan->host_tensors.assign(ht, ht + num_tensors);
    plan->chunk_start.swap(chunk_start);
    if (hipMalloc(&plan->device_block, total) != hipSuccess) {
        (void)hipGetLastError();
        plan->device_block = nullptr;
        return CDSGD_ERR_DEVICE;
    }
    if (hipMemcpy(plan->device_block, image.data(), total, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        return CDSGD_ERR_DEVICE;
    }
    unsigned char *base = static_cast<unsigned char *>(plan->device_block);
    plan->tensors = reinterpret_cast<TensorDesc *>(base);
    plan->chunks = reinterpret_cast<ChunkRef *>(base + off_c);
    plan->rows = reinterpret_cast<const uint8_t **>(base + off_p);
    if (arenas) plan->arena_chunks = reinterpret_cast<ArenaChunk *>(base + off_a);
    plan->num_tensors = num_tensors;
    plan->num_workers = num_workers;
    plan->self = self;
    plan->num_chunks = (unsigned)total_chunks;
    plan->has_agg_full = all_agg;
    plan->grad_type = grad_dtype;
    *out = plan.release();
    return CDSGD_OK;
} catch (const std::bad_alloc &) {
    return CDSGD_ERR_DEVICE;
}

int cdsgd_plan_destroy(cdsgd_plan *plan)
{
    if (!plan) return CDSGD_OK;
    int rc = CDSGD_OK;
    if (plan->device_block && hipFree(plan->device_block) != hipSuccess) {
        (void)hipGetLastError();
        rc = CDSGD_ERR_DEVICE;
    }
    if (plan->peer_grads_block && hipFree(plan->peer_grads_block) != hipSuccess) {
        (void)hipGetLastError();
        rc = CDSGD_ERR_DEVICE;
    }
    delete plan;
    return rc;
}

namespace {

// Launch shape of a compressed pass: waves per group, the LDS a group asks for in all (0: what it uses), and whether the
// workers' words are asked for behind the tile's own streams instead of in front of them.
//
// The passes are bound by HBM, and HBM serves a mix of reads and writes best when the streams' requests in flight
// stay close together: groups are dispatched in order, so the number of groups resident bounds how far apart they
// are, and the LDS that a group asks for bounds that number (160 KiB per compute unit).  Short lists fit the
// memory-side cache in part and end before such an order matters: there every resident group helps.  Words asked for
// first are there soonest for the decode (ResNet-50-shaped list in ranges of a million elements, N = 16: 166.5 us
// against 169.3), asked for last they leave the order of the tile's own streams at HBM alone.
//
// Measured: time of the pass over that of the kernels before these (one 128-bit load for 16 peers, bytes staged
// through LDS), with several sets of buffers in turn (5 GB in all, as a program that does something else between two
// passes leaves the memory-side cache).  Lists: flat of 20, 40 and 90 M elements, VGG-16-shaped.  Groups per compute
// unit, "all" where registers alone bound them; "late": words last.
//   up to 8 workers, one-wave groups    all / 26 / 22 / 20              four waves: all / 3
//     N = 4, t = 0.3, 32-bit   20 M     .99 / .99 / .99 / .99           1.01 / .99
//                              90 M    1.03 / 1.04 / 1.00 / 1.00        1.08 / .99
//                              VGG-16  1.03 / 1.04 / 1.00 / .98         1.10 / .95
//     N = 4, t = 0.3, bf16     40 M    1.01 / 1.00 / .99 / 1.00         1.04 / 1.00
//     N = 8, t = 0.3, bf16     40 M    1.02 / 1.02 / 1.00 / 1.00        1.04 / 1.00     (25 M, fp16: 94.9 us with 26, 95.5 with 22)
//                              VGG-16  1.05 / 1.04 / 1.00 / 1.01        1.08 / 1.01
//     N = 8, t = 0.5, 32-bit   40 M    1.01 / 1.01 / .99 / .98          1.04 / .98
//                              VGG-16  1.05 / 1.05 / 1.03 / 1.00        1.12 / .99
//   9 to 16 workers, count form         all / 5 / 4 / 3                 late: all / 5 / 4 / 3
//     N = 16, 32-bit           20 M    1.03 / .98 / .99 / .97           1.04 / .98 / .98 / .97
//                              40 M    1.04 / 1.01 / 1.00 / .98         1.04 / .99 / .99 / .98
//                              VGG-16  1.09 / 1.03 / 1.02 / .99         1.10 / 1.02 / 1.03 / .98
//     N = 16, bf16             20 M    1.00 / .96 / .96 / .97           .98 / .96 / .97 / 1.00
//                              40 M    1.03 / .98 / .97 / .98           1.02 / .98 / .97 / 1.01
//                              VGG-16  1.05 / .98 / .98 / .98           1.04 / .97 / .97 / 1.01
//   9 to 16 workers, chain form         all / 5 / 3                     late: all / 5
//     N = 16, t = 0.3, 32-bit  26 M    1.01 / 1.00 / 1.07               1.00 / 1.01
//                              40 M    1.02 / .99 / 1.05                1.02 / 1.00
//                              VGG-16  1.09 / 1.00 / 1.06               1.08 / 1.01
//     N = 16, t = 0.3, bf16    40 M    1.00 / 1.00 / 1.07               .99 / 1.00
//                              VGG-16  1.03 / 1.01 / 1.07               1.02 / 1.00
//   above 16 workers                    all / 5 / 3
//     N = 32, t = 0.5, 32-bit  20 M    1.02 / 1.00 / 1.00
//                              VGG-16  1.06 / 1.01 / 1.00
//     N = 32, t = 0.3, 32-bit  20 M    .98 / .94 / 1.00                 (VGG-16: 1.01 / .95 / 1.04)
//     N = 17, t = 0.3, bf16    26 M    1.01 / 1.02 / 1.17               (VGG-16: 1.05 / 1.01 / 1.16)
//   sparse peers                        all / 5       one code in 256, then one in 4
//     N = 8, t = 0.3           VGG-16  1.01 / .98     1.04 / .97
//     N = 9 / 16, t = 0.5      VGG-16   .97 / 1.01, .97 / .99     1.00 / .98, 1.03 / 1.01
//     N = 16, t = 0.3          VGG-16   .88 / .99     .93 / 1.01
//   (The bound of the sparse count form above 8 workers costs 3 % where few codes are sent and saves as much where many are.)
// Six groups (kSix) where the kernels' registers would admit seven or eight ("all" above is six in those rows: they held more
// scalar registers then).  Time over that of six, 7 groups / 6:
//   9 to 16 workers, chain    N = 9, 12, 16, t = 0.1  bf16 20 M 1.01-1.02 / 1, 40 M 1.02-1.03, 60 M 1.02-1.04, 32-bit 25 M 1.00
//   the same, sparse          one code in 16  25 M .99-1.01, 60 M 1.00-1.03, VGG-16-shaped 1.04-1.07, 260 M 1.06-1.09, bf16 138 M 1.05-1.08
//                             (below 16 M six take longer: 2 M 1.05, 4 M 1.01-1.04)
//   17 to 32 workers, sparse  138 M, bf16  N = 17 / 20 1.04 / 1.01-1.03, t = 0.5 1.02 / 1.02, N = 32 .99-1.00;  60 M 1.00, N = 32 .99  (18 to 25 M .99: no bound there)
//   up to 8 workers, sparse   18 M, t = 0.1  N = 4 1.000, N = 8 1.006;  25 M N = 4 1.005, N = 8 1.015;  t = 0.5 1.00;  ResNet-50-shaped,
//                             t = 0.5, N = 8 1.01, one code in 256, bf16 1.006-1.008
//   9 to 16 workers, sparse, t = 0.5   18 and 25 M 1.00;  ResNet-50-shaped 1.00, one code in 256, bf16 1.003-1.006
//   (Above 32 workers the registers admit six.)
// Five groups over six, 16-bit chains: N = 9 / 12 / 13 / 16  50 M 1.03 / 1.02 / .98 / .98, 80 M .99 / .99 / .98-.99 / .98;  17 to 32 workers, 18 to
// 25 M  N = 24 .98-1.02, N = 28 / 30 / 32 .98-.99 / .97 / .96, ResNet-50-shaped .98 / 1.00 / .96.
// The same buffers pass after pass with nothing in between are another matter: up to 64 M elements part of them is
// still in the memory-side cache, and lists of 28 to 64 M elements of 9 to 16 workers would run up to 7 % faster with
// all groups (N = 16, t = 0.3, 64 M: 267 us, 284 with 5).  No training step leaves the cache alone like that.
//
// With a workgroup limit the groups walk the list, and drift apart as they go: the more of them, the farther apart the
// streams' requests.  Three to a compute unit keep HBM busy, so above 16 M elements a larger limit is not used up;
// groups of four waves whatever the length, so that a limit means the same everywhere; 32 KiB each, which leaves 64 of
// a compute unit's 160 to kernels that run beside (the former kernels held 16 KiB for each of up to five groups) and
// keeps a kernel that fills the chip from starving the pass.  VGG-16-shaped, us: the former kernels / as many groups
// as the limit allows, none bounded / now:
//   alone, N = 16, t = 0.5     limit 1024 711 / 789 / 712;  2048 748 / 801 / 712;  4096 777 / 855 / 712
//   alone, N = 16, t = 0.3     1024 717 / 775 / 693;  4096 776 / 839 / 693
//   alone, N = 32, t = 0.5     1024 831 / 909 / 839;  4096 825 / 987 / 839
//   alone, N = 4, t = 0.5      512 1942 / 1671 / 549 (one-wave groups before);  4096 632 / 640 / 566
//   the other half of the split step alone, N = 16: 1024 576 / 659 / 617;  2048 607 / 665 / 613;  t = 0.3, 1024
//   606 / 624 / 567  (behind the former kernels at t = 0.5 and limits near 1024: two groups per compute unit take
//   520 us alone, but beside the small products below 1620 us against 1250, so three stay)
//   the other half of the split step in a stream beside 48 small products, N = 16: 2048 1282 / 1406 / 1275;
//   N = 8: 4096 1135 / 1340 / 1175;  beside one product that fills the chip, N = 16: 2048 1706 / 1732 / 1742 (1906
//   without the LDS);  N = 8: 4096 1656 / 1705 / 1665
// The exceptions: a limit of more than a sixth of the tiles hardly limits, and the pass has the LDS that it has without
// one (N = 16, limit 60000: 687 us with no bound, 668); sparse streams drift less and use the limit up (N = 16, t = 0.3,
// 25 M elements, 8192: 112 us, 122 with 768 groups), but for the long lists of the count form (4096: 673 and 650).
// The words are asked for last where that is better: 16-bit gradients (N = 16, limit 700: 647 us, 708 with the words
// first), 32-bit ones up to 512 groups (25 M elements 117 and 121; 768 groups, VGG-16-shaped, 757 and 712).
constexpr unsigned kWalkingGroups = 768;

// Stores and the loads of the words.  Non-temporal stores leave dirty lines in the L2s of the compute dies, the packed
// codes' at the default policy all of them, for the flush at the end of the kernel; written through they leave none.
// Time of the pass with results written through over that without:
//   9 to 16 workers   N = 9 / 12 / 16 count, 16 chain, 16 chain bf16   2 M .99 / - / .99 / .99 / .97;  12 M - / .99 / - /
//                     .99 / .98;  18 M 1.00 / - / .98 / 1.00 / .99;  25 M - / .99 / .97 / .97 / .98;  40 M .98 / - / .98 /
//                     .99 / .98;  VGG-16 - / .99 / .99 / 1.00 / .98;  90 M 1.04 / - / .99 / 1.01 / .99;  260 M .99 / - /
//                     .99 / 1.00 / .98   (long 32-bit chains gain nothing and 1 GiB buckets at t = 0.05 lose 1 %)
//   (Where the buffers lie moves long lists by more than that.  Count form, 32-bit, lowest - highest, mean over 8 to 20 lengths
//   and places:  30 to 60 M elements N = 9 to 12 .96 - .99, .98;  13 to 16 .95 - 1.00, .98;  64 to 150 M N = 9 .95 - 1.05, .99;
//   10 .96 - 1.06, .99;  11 .98 - 1.04, .99;  12 .94 - 1.09, 1.00;  13 .97 - 1.03, .99;  14 to 16 .97 - 1.00, .99.  Non-temporal stores
//   for 9 to 12 workers above 60 M take the worst places back and cost 1 % in the mean.)
//   (short lists, whose results the next pass finds in a cache, are slower so: N = 9 / 16, t = 0.3, bf16 0.3 M 1.16 / 1.16,
//   0.45 M 1.24 / 1.23, 0.7 M 1.14 / 1.07, 1 M .98 / .98, 1.4 M 1.00 / .99;  N = 17 / 32 0.45 M 1.15 / 1.07, 1 M 1.04 / 1.07,
//   1.4 M 1.03 / 1.01;  32-bit, t = 0.3, N = 16 / 32 0.45 M 1.10 / 1.00, 1 M .99 / 1.05, 1.4 M 1.02 / 1.02)
//   up to 8 workers   N = 4, t = 0.3  4 M 1.03, 12 M .99, 25 M 1.00, VGG-16 1.06;  N = 8 1.02 / 1.00 / 1.01 / 1.00
// Kernels of their own for 17 to 32 workers, whose waves hold half as many stream pointers, over those for any number (results
// written through / and the list in arenas), N = 17 / 24 / 32:
//   t = 0.5, 32-bit   1 M .83 .83 .88 / .81 .82 .88;  4 M .98 .97 .98 / .98 .97 .97;  12 M .99 .99 .98 / .99 .99 .99;
//                     ResNet-50-shaped .97 .98 .98 / .97 .97 .98;  VGG-16 .99 1.00 1.01
//   t = 0.3, 32-bit   1 M .97 1.03 .97 / .93 .99 .96;  4 M .99 .99 1.00 / .98 .98 .98;  12 M 1.00 .99 .97 / .99 .99 .99;
//                     ResNet-50-shaped .95 .97 .97 / .95 .95 .96;  VGG-16 .98 1.01 1.00
//   t = 0.3, bf16     1 M .88 .94 1.02 / .88 .93 1.03;  4 M .99 / .98;  12 M 1.00 1.00 .98 / .99 .98 .98;  VGG-16 .96 .98 1.00
// (Long 32-bit lists of more than 20 workers keep the general kernels.)
// Words read non-temporally, as in decode-and-sum, and 5 groups, over the default policy at its own residency:
//   N = 33   8 M 1.07-1.08, 20 M .97-1.00, 50 M .96;  N = 48  8 M 1.06, 10 M .96;  N = 64  6 M 1.04, 8 M .95, 25 M .96-.98,
//   VGG-16 .94-.99   (N = 17: 25 M .99-1.03, VGG-16 1.00-1.04;  N = 32: 25 M .98-.99, VGG-16 1.02-1.04;  N = 16 25 M 1.04)
constexpr unsigned long long kStreamWordsBytes = 112000000;

// Lists in arenas (ArenaChunk), up to 32 workers and 28 M elements: one trip to memory less before a group's first data
// loads.  Time over that of the general kernels: 1 M elements .97-1.00, 2 M .97-.99, 4 M .98-.99, 8 M .99-1.00, 25 M
// .99-1.01; ResNet-50-shaped list, N = 16, in 19 launches of a million elements and more 163.1 / 156.9 us, in one 107.0 /
// 106.2;  N = 32, t = 0.5 / 0.1 / 0.1 in bf16  0.3 M .92 / .99 / .99, 0.9 M .95 / .96 / .97, 1.5 M .97 / .99 / .98, 3 M .98 / .98 / .97,
// 8 M .99 / 1.00 / .99, 20 M 1.00 / 1.00 / .99, 26 M 1.01 / 1.00 / 1.00.  (VGG-16-shaped .99-1.04, 1 GiB buckets 1.02.  Above 32
// workers 1 M 1.12, 4 M 1.03, 25 M 1.01, in kernels that held the pointers, more than there are scalar registers, through the loop over tiles.)
constexpr int kUpTo32Rows = 16;  // host side only: the kernels for up to 32 workers
struct CompressedLaunch {
    unsigned waves, lds;
    int how;          // kLate, kWrittenOut, kStreamWords, kArena, kSixGroups, kFewGroups, kUpTo32Rows
    unsigned groups;  // launch at most this many (0: no bound)
};

CompressedLaunch compressed_launch(unsigned num_chunks, int num_workers, int form, bool sparse, bool arenas, int grad_type,
                                   unsigned max_workgroups)
{
    const unsigned tiles = num_chunks * kTilesPerChunk;  // of 1024 elements
    const bool mid_list = tiles > kMidListTiles, long_list = tiles > kLongListTiles, half = grad_type != kGradF32;
    if (max_workgroups != 0) {
        const bool walk = max_workgroups <= tiles / 6u, count16 = form == kCount && num_workers > kUpTo8 && num_workers <= kUpTo16;
        // Up to 8 workers, few groups that walk the list, each waiting for the last of its loads.  Since ragged ends are read without tests
        // the compiler asks for the words behind gradient and residual; the chain's rows it reads in two trips.  Time over that with the
        // tests, in the compiler's order / so, 16 to 256 groups:  count form, 32-bit  N = 2 to 8, 4 to 70 M 1.002-1.007 / .97-.99;  chain  N = 5 and 8
        // 1.014-1.020 / .98-.99, 16-bit 1.00-1.01 / .98-.99, N = 2 and 4 .99 / .985-.99;  both, 0.3 M, 64 groups 1.00-1.03 / .96-1.00.  (Count form,
        // 16-bit, stays as it is, 1.004-1.019: so, 4 and 20 M .94-1.00, but 70 M 1.07-1.08.  More groups: .99-1.01 either way.)
        const bool few = !sparse && num_workers <= kUpTo8 && max_workgroups <= tiles / 2u && (form == kChain || (form == kCount && !half));
        const int few_groups = few ? kFewGroups : 0;
        if (!mid_list || (sparse && !(walk && long_list && count16))) return {4u, 0u, few_groups, 0u};
        if (walk) return {4u, 32768u, few_groups | (!sparse && count16 && (half || max_workgroups <= 512u) ? kLate : 0), kWalkingGroups};
        if (num_workers <= kUpTo8) return {4u, 49152u, 0, 0u};
    }
    if (form == kChainTiny) {
        const bool all = !long_list || (sparse && num_workers > kUpTo16);
        return {4u, all ? 0u : (num_workers <= kUpTo16 ? 32768u : 38912u), 0, 0u};
    }
    if (sparse) {
        const bool five = long_list && (num_workers <= kUpTo8 || (num_workers <= kUpTo16 && form == kCount));
        const bool six = num_workers <= kUpTo16 ? mid_list : long_list && half && num_workers <= kUpTo32;
        return {4u, five ? 32768u : 0u, six && !five ? kSixGroups : 0, 0u};
    }
    const int arena = arenas && max_workgroups == 0 ? kArena : 0;
    const int out = tiles > (num_workers <= kUpTo16 ? 1024u : 2048u) ? kWrittenOut : 0;
    if (num_workers <= kUpTo8) {
        if (!mid_list) return {4u, 0u, arena, 0u};
        if (tiles <= 48u * 1024u) return {1u, half && !long_list ? 6144u : 7168u, long_list ? 0 : arena, 0u};
        if (num_workers > 4) return {4u, 49152u, 0, 0u};
        return {1u, half ? 7168u : 8192u, 0, 0u};
    }
    if (num_workers <= kUpTo16 && form == kCount) {
        if (tiles <= 6u * 1024u) return {4u, 0u, out | arena, 0u};
        if (!mid_list) return {4u, 24576u, kWrittenOut | arena, 0u};
        if (half) return {4u, 40960u, kWrittenOut | (long_list ? 0 : arena), 0u};
        if (long_list) return {4u, 49152u, kWrittenOut | kLate, 0u};
        return {4u, 32768u, kWrittenOut | kLate | arena, 0u};
    }
    if (num_workers <= kUpTo16) {
        if (tiles > (half ? (num_workers > 12 ? 48u : 80u) * 1024u : kLongListTiles))
            return {4u, 32768u, half || tiles <= 48u * 1024u ? kWrittenOut : 0, 0u};
        return {4u, 0u, out | (mid_list ? kLate : 0) | (long_list ? 0 : arena), 0u};
    }
    if (num_workers <= kUpTo32 && max_workgroups == 0 && (half || !long_list || num_workers <= 20)) {
        const bool bounded = half && form != kCount && num_workers < 28 ? long_list : mid_list;
        return {4u, !bounded ? 0u : (form == kCount ? 32768u : 38912u), kUpTo32Rows | out | (long_list ? 0 : arena), 0u};
    }
    if (num_workers > kUpTo32 && (unsigned long long)num_workers * tiles * kTileBytes > kStreamWordsBytes)
        return {4u, 32768u, kStreamWords, 0u};
    if (form == kCount) return {4u, mid_list ? 32768u : 0u, 0, 0u};
    return {4u, (half ? long_list : mid_list) ? 38912u : 0u, 0, 0u};
}

// The launch of a compressed pass over a plan's tables with the call's threshold, and the form of its decode.
CompressedLaunch launch_of_pass(const PlanTables *plan, float threshold, int *form)
{
    // the count form of the decode needs every threshold in use to be a power of two; the chain form's multipliers
    // need half of each to be exact
    const bool pow2 = plan->own_thresholds ? plan->own_thresholds_pow2 : is_pow2_threshold(threshold);
    const bool tiny = plan->own_thresholds ? plan->own_thresholds_tiny : is_tiny_threshold(threshold);
    *form = pow2 ? kCount : (tiny ? kChainTiny : kChain);
    return compressed_launch(plan->num_chunks, plan->num_workers, *form, plan->peers_sparse, plan->has_arenas(), plan->grad_type,
                             plan->max_workgroups);
}

// One pass of FormalTraining's loop; with_local = false leaves eq. 11 out (split form).
int launch_formal_pass(const PlanTables *plan, long step, int k, float threshold, float lr_local, float lr_global,
                       bool with_local, void *hip_stream)
{
    if (!plan) return CDSGD_ERR_NULL;
    if (!good_step_params(step, k, threshold, lr_local, lr_global)) return CDSGD_ERR_PARAM;
    const bool compressed = (step % k) != 0;
    if (!compressed)
        return launch_full_pass(plan, with_local ? kLocalRule : kLocalNone, lr_local, lr_global, hip_stream);
    const float scale = lr_global / (float)plan->num_workers;
    hipStream_t s = (hipStream_t)hip_stream;
    const int N = plan->num_workers;
    int form;
    const CompressedLaunch shape = launch_of_pass(plan, threshold, &form);
    const unsigned num_tiles = plan->num_chunks * (kChunkQuads / (64u * shape.waves));
    unsigned grid = plan->grid_size(num_tiles, 64u * shape.waves);
    if (shape.groups != 0 && grid > shape.groups) grid = shape.groups;
    // Sparse peers of 17 to 32 workers: the kernels for so many over those for any number, N = 17 / 24 / 32: t = 0.5 1 M 1.01 /
    // 1.03 / .99, 4 M .97, ResNet-50-shaped .98;  t = 0.3 1 M .91 / .96 / .98, 4 M .94, ResNet-50-shaped .95 / .98 / .98,
    // VGG-16-shaped 1.00 / 1.03 / 1.00;  t = 0.3, bf16 1 M .90 / .91 / .92, 4 M .93, VGG-16-shaped .94 / .97 / .98.
    const bool sparse32 = N <= kUpTo32 && plan->max_workgroups == 0 &&
                          (plan->grad_type != kGradF32 || plan->num_chunks * kTilesPerChunk <= kLongListTiles);
    // Passes in which the weights are asked for behind gradient and residual.  Time over that of asking for all at once:
    // 17 to 32 workers, lists of 2 to 16 M elements in arenas, written through, six and three sets of buffers in turn, 2.2 / 3 / 5 / 8 / 12 / 16 M:
    //   t = 0.1  N = 17 .97 .98 .99 .99 .99 .99;  20 .97 .98 .99 1.00 .99 .99;  24 .98 .98 .99 .99 .99 .99;  32 .98 .98 .99 .99 1.00 .99
    //   t = 0.1, bf16  N = 17 .99 .99 .99 .99 .99 .99;  20 1.00 .99 .99 .99 1.00 .99;  24 .99 .99 .99 .99 .99 1.00;  32 1.00 .99 1.00 1.00 1.00 1.01
    //   t = 0.5  N = 17 1.01 1.00 1.00 1.00 .99 .99;  20 1.01 1.00 1.00 1.00 1.00 .99;  24 1.00 1.00 1.01 1.00 .99 1.00;  32 1.00 1.00 1.00 1.00 1.00 1.00
    //   (25 M 1.00-1.02;  9 to 16 workers, t = 0.5: 1.1 M .96, 1.5 M 1.02, 3 M 1.01, 8 to 16 M .99, 25 M 1.01, 25 M in bf16 1.03)
    // Count form above 32 workers, words read non-temporally, 9 / 14 / 18 / 26 / 40 / 64 / 100 M:
    //   32-bit  N = 33 1.00 .99 .98 1.00 .99 1.00 1.00;  48 1.00 .99 1.00 1.00 1.00 .99 1.00;  64 .99 .99 .99 .99 1.00 .99 1.00
    //   bf16    N = 33 1.00 .99 1.00 1.00 1.00 .99 .99;  48 1.00 .99 .99 .99 1.00 .99 .99;  64 .98 .99 .99 .99 1.00 .99 .99
    //   (the chain there: .99-1.01)
    const bool weights_wait = plan->num_chunks * kTilesPerChunk <= kMidListTiles;
    const auto bound = [&](unsigned used) { return shape.lds <= used ? 0u : shape.lds - used; };
#define CDSGD_LAUNCH_COMPRESSED_S(SZ, WAVES, FORM, GT, SPARSE, HOW, WAIT)                                      \
    hipLaunchKernelGGL((k_fused_compressed<SZ, WAVES, FORM, GT, SPARSE, HOW, WAIT>), dim3(grid), dim3(64 * WAVES), \
                       bound(kTileLds<SZ, FORM, WAVES, SPARSE, true>), s, plan->tensors, plan->table_for<HOW>(), plan->rows, \
                       num_tiles, grid, N, plan->self, threshold, lr_local, scale, with_local ? 1 : 0)
#define CDSGD_LAUNCH_COMPRESSED_W(SZ, WAVES, FORM, SPARSE, HOW, WAIT)                                          \
    do {                                                                                                       \
        if (plan->grad_type == kGradBF16) CDSGD_LAUNCH_COMPRESSED_S(SZ, WAVES, FORM, kGradBF16, SPARSE, HOW, WAIT); \
        else if (plan->grad_type == kGradF16) CDSGD_LAUNCH_COMPRESSED_S(SZ, WAVES, FORM, kGradF16, SPARSE, HOW, WAIT); \
        else CDSGD_LAUNCH_COMPRESSED_S(SZ, WAVES, FORM, kGradF32, SPARSE, HOW, WAIT);                          \
    } while (0)
#define CDSGD_LAUNCH_COMPRESSED(SZ, WAVES, FORM, SPARSE, HOW) CDSGD_LAUNCH_COMPRESSED_W(SZ, WAVES, FORM, SPARSE, HOW, false)
// (the count form asks for the words last, 9 to 16 workers, or first, few groups, with 32-bit gradients only: compressed_launch)
#define CDSGD_LAUNCH_COMPRESSED_32BIT(SZ, WAVES, FORM, SPARSE, HOW)                                            \
    do {                                                                                                       \
        if (plan->grad_type != kGradF32) return CDSGD_ERR_DEVICE;                                              \
        CDSGD_LAUNCH_COMPRESSED_S(SZ, WAVES, FORM, kGradF32, SPARSE, HOW, false);                              \
    } while (0)
#define CDSGD_LAUNCH_COMPRESSED_16BIT(SZ, WAVES, FORM, SPARSE, HOW)                                            \
    do {                                                                                                       \
        if (plan->grad_type == kGradBF16) CDSGD_LAUNCH_COMPRESSED_S(SZ, WAVES, FORM, kGradBF16, SPARSE, HOW, false); \
        else if (plan->grad_type == kGradF16) CDSGD_LAUNCH_COMPRESSED_S(SZ, WAVES, FORM, kGradF16, SPARSE, HOW, false); \
        else return CDSGD_ERR_DEVICE;                                                                          \
    } while (0)
// Every shape has a kernel of its own; one that has none is an error, for another kernel may read the tables otherwise.
#define CDSGD_LAUNCH_COMPRESSED_F(FORM, LAUNCH_LATE)                                                           \
    do {                                                                                                       \
        if (plan->peers_sparse && shape.how != 0 && shape.how != kSixGroups) return CDSGD_ERR_DEVICE;          \
        else if (shape.how == kSixGroups && (!plan->peers_sparse || N > kUpTo32)) return CDSGD_ERR_DEVICE;     \
        else if (shape.how == kSixGroups && N <= kUpTo8) CDSGD_LAUNCH_COMPRESSED(kUpTo8, 4, FORM, true, kSixGroups); \
        else if (shape.how == kSixGroups && N <= kUpTo16) CDSGD_LAUNCH_COMPRESSED(kUpTo16, 4, FORM, true, kSixGroups); \
        else if (shape.how == kSixGroups) CDSGD_LAUNCH_COMPRESSED_16BIT(kUpTo32, 4, FORM, true, kSixGroups);   \
        else if (plan->peers_sparse && N <= kUpTo8) CDSGD_LAUNCH_COMPRESSED(kUpTo8, 4, FORM, true, 0);         \
        else if (plan->peers_sparse && N <= kUpTo16) CDSGD_LAUNCH_COMPRESSED(kUpTo16, 4, FORM, true, 0);       \
        else if (plan->peers_sparse && sparse32) CDSGD_LAUNCH_COMPRESSED(kUpTo32, 4, FORM, true, 0);           \
        else if (plan->peers_sparse) CDSGD_LAUNCH_COMPRESSED(kAnyWorkers, 4, FORM, true, 0);                   \
        else if (shape.waves == 1u && shape.how == kArena) CDSGD_LAUNCH_COMPRESSED(kUpTo8, 1, FORM, false, kArena); \
        else if (shape.waves == 1u && shape.how == 0) CDSGD_LAUNCH_COMPRESSED(kUpTo8, 1, FORM, false, 0);      \
        else if (N <= kUpTo8 && shape.how == kArena) CDSGD_LAUNCH_COMPRESSED(kUpTo8, 4, FORM, false, kArena);  \
        else if (N <= kUpTo8 && shape.how == kFewGroups) LAUNCH_LATE(kUpTo8, 4, FORM, false, kFewGroups); \
        else if (N <= kUpTo8 && shape.how == 0) CDSGD_LAUNCH_COMPRESSED(kUpTo8, 4, FORM, false, 0);            \
        else if (N <= kUpTo8) return CDSGD_ERR_DEVICE;                                                         \
        else if (shape.how == (kUpTo32Rows | kWrittenOut | kArena) && weights_wait) CDSGD_LAUNCH_COMPRESSED_W(kUpTo32, 4, FORM, false, kWrittenOut | kArena, true); \
        else if (shape.how == (kUpTo32Rows | kWrittenOut | kArena)) CDSGD_LAUNCH_COMPRESSED(kUpTo32, 4, FORM, false, kWrittenOut | kArena); \
        else if (shape.how == (kUpTo32Rows | kWrittenOut)) CDSGD_LAUNCH_COMPRESSED(kUpTo32, 4, FORM, false, kWrittenOut); \
        else if (shape.how == (kUpTo32Rows | kArena)) CDSGD_LAUNCH_COMPRESSED(kUpTo32, 4, FORM, false, kArena); \
        else if (shape.how == kUpTo32Rows) CDSGD_LAUNCH_COMPRESSED(kUpTo32, 4, FORM, false, 0);                \
        else if (N > kUpTo16 && shape.how == kStreamWords) CDSGD_LAUNCH_COMPRESSED_W(kAnyWorkers, 4, FORM, false, kStreamWords, FORM == kCount); \
        else if (N > kUpTo16 && shape.how == 0) CDSGD_LAUNCH_COMPRESSED(kAnyWorkers, 4, FORM, false, 0);       \
        else if (N > kUpTo16) return CDSGD_ERR_DEVICE;                                                         \
        else if (shape.how == (kWrittenOut | kLate | kArena)) LAUNCH_LATE(kUpTo16, 4, FORM, false, kWrittenOut | kLate | kArena); \
        else if (shape.how == (kWrittenOut | kLate)) LAUNCH_LATE(kUpTo16, 4, FORM, false, kWrittenOut | kLate); \
        else if (shape.how == (kWrittenOut | kArena)) CDSGD_LAUNCH_COMPRESSED(kUpTo16, 4, FORM, false, kWrittenOut | kArena); \
        else if (shape.how == kWrittenOut) CDSGD_LAUNCH_COMPRESSED(kUpTo16, 4, FORM, false, kWrittenOut);      \
        else if (shape.how == kArena) CDSGD_LAUNCH_COMPRESSED(kUpTo16, 4, FORM, false, kArena);                \
        else if (shape.how == 0) CDSGD_LAUNCH_COMPRESSED(kUpTo16, 4, FORM, false, 0);                          \
        else return CDSGD_ERR_DEVICE;                                                                          \
    } while (0)
    if (form == kChainTiny && shape.how != 0) return CDSGD_ERR_DEVICE;
    if (form == kCount && shape.how == kLate) CDSGD_LAUNCH_COMPRESSED(kUpTo16, 4, kCount, false, kLate);  // walking groups
    else if (form == kCount) CDSGD_LAUNCH_COMPRESSED_F(kCount, CDSGD_LAUNCH_COMPRESSED_32BIT);
    else if (form == kChain) CDSGD_LAUNCH_COMPRESSED_F(kChain, CDSGD_LAUNCH_COMPRESSED);
    else if (plan->peers_sparse) CDSGD_LAUNCH_COMPRESSED(kAnyWorkers, 4, kChainTiny, true, 0);
    else CDSGD_LAUNCH_COMPRESSED(kAnyWorkers, 4, kChainTiny, false, 0);
#undef CDSGD_LAUNCH_COMPRESSED_32BIT
#undef CDSGD_LAUNCH_COMPRESSED_16BIT
#undef CDSGD_LAUNCH_COMPRESSED
#undef CDSGD_LAUNCH_COMPRESSED_W
#undef CDSGD_LAUNCH_COMPRESSED_F
#undef CDSGD_LAUNCH_COMPRESSED_S
    return launch_status();
}

}  // namespace

int cdsgd_step_fused(cdsgd_plan *plan, long step, int k, float threshold, float lr_local, float lr_global,
                     void *hip_stream)
{
    return launch_formal_pass(plan, step, k, threshold, lr_local, lr_global, true, hip_stream);
}

namespace {

// eq. 11 alone over the chunks a PlanTables covers.
int launch_local_pass(const PlanTables *plan, float lr_local, void *hip_stream)
{
    if (!plan) return CDSGD_ERR_NULL;
    if (!std::isfinite(lr_local)) return CDSGD_ERR_PARAM;
    const unsigned long long num_pieces = (unsigned long long)plan->num_chunks * kPiecesPerChunk;
    const dim3 grid(plan->grid_size(num_pieces, kFullBlock)), block(kFullBlock);
    hipStream_t s = (hipStream_t)hip_stream;
#define CDSGD_LAUNCH_LOCAL(GT)                                                                                 \
    hipLaunchKernelGGL((k_fused_full<false, kLocalOnly, GT, kStream, kInOrder>), grid, block, 0, s, plan->tensors,                  \
                       plan->chunk_table(), num_pieces, (const void *const *)nullptr, 0, plan->self, lr_local,   \
                       0.0f)
    if (plan->grad_type == kGradBF16) CDSGD_LAUNCH_LOCAL(kGradBF16);
    else if (plan->grad_type == kGradF16) CDSGD_LAUNCH_LOCAL(kGradF16);
    else CDSGD_LAUNCH_LOCAL(kGradF32);
#undef CDSGD_LAUNCH_LOCAL
    return launch_status();
}

// The part of a plan's tables that covers tensors [first_tensor, first_tensor + num_tensors).
int slice_of_plan(const cdsgd_plan *plan, int first_tensor, int num_tensors, PlanTables *out)
{
    if (!plan) return CDSGD_ERR_NULL;
    if (first_tensor < 0 || num_tensors < 1 || first_tensor > plan->num_tensors - num_tensors) return CDSGD_ERR_PARAM;
    *out = *plan;  // the tables themselves are shared; only the range of chunks differs
    out->first_chunk = plan->chunk_start[(size_t)first_tensor];
    out->num_chunks = plan->chunk_start[(size_t)first_tensor + (size_t)num_tensors] - out->first_chunk;
    return CDSGD_OK;
}

}  // namespace

int cdsgd_step_local(cdsgd_plan *plan, float lr_local, void *hip_stream)
{
    return launch_local_pass(plan, lr_local, hip_stream);
}

int cdsgd_step_global(cdsgd_plan *plan, long step, int k, float threshold, float lr_global, void *hip_stream)
{
    return launch_formal_pass(plan, step, k, threshold, 0.0f, lr_global, false, hip_stream);
}

int cdsgd_step_fused_range(cdsgd_plan *plan, int first_tensor, int num_tensors, long step, int k, float threshold,
                           float lr_local, float lr_global, void *hip_stream)
{
    PlanTables part;
    const int rc = slice_of_plan(plan, first_tensor, num_tensors, &part);
    if (rc != CDSGD_OK) return rc;
    return launch_formal_pass(&part, step, k, threshold, lr_local, lr_global, true, hip_stream);
}

int cdsgd_step_local_range(cdsgd_plan *plan, int first_tensor, int num_tensors, float lr_local, void *hip_stream)
{
    PlanTables part;
    const int rc = slice_of_plan(plan, first_tensor, num_tensors, &part);
    if (rc != CDSGD_OK) return rc;
    return launch_local_pass(&part, lr_local, hip_stream);
}

int cdsgd_step_global_range(cdsgd_plan *plan, int first_tensor, int num_tensors, long step, int k, float threshold,
                            float lr_global, void *hip_stream)
{
    PlanTables part;
    const int rc = slice_of_plan(plan, first_tensor, num_tensors, &part);
    if (rc != CDSGD_OK) return rc;
    return launch_formal_pass(&part, step, k, threshold, 0.0f, lr_global, false, hip_stream);
}

int cdsgd_plan_bind_full_grads(cdsgd_plan *plan, const float *const *const *peer_grads)
try {
    if (!plan) return CDSGD_ERR_NULL;
    const int np = plan->num_workers - 1;
    if (np == 0) return CDSGD_OK;  // a single worker's sum is its own gradient
    if (!peer_grads) return CDSGD_ERR_NULL;
    std::vector<const void *> image((size_t)plan->num_tensors * (size_t)np);
    for (int j = 0, slot = 0; j < plan->num_workers; ++j) {
        if (j == plan->self) continue;
        if (!peer_grads[j]) return CDSGD_ERR_NULL;
        for (int i = 0; i < plan->num_tensors; ++i) {
            if (!peer_grads[j][i]) return CDSGD_ERR_NULL;
            if (!aligned(peer_grads[j][i], 16)) return CDSGD_ERR_ALIGN;
            image[(size_t)i * (size_t)np + (size_t)slot] = peer_grads[j][i];
        }
        ++slot;
    }
    const size_t bytes = image.size() * sizeof(const void *);
    void *dev = plan->peer_grads_block;
    if (!dev && hipMalloc(&dev, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return CDSGD_ERR_DEVICE;
    }
    if (hipMemcpy(dev, image.data(), bytes, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        if (!plan->peer_grads_block) (void)hipFree(dev);
        return CDSGD_ERR_DEVICE;
    }
    plan->peer_grads_block = dev;
    plan->peer_grads = (const void **)dev;
    return CDSGD_OK;
} catch (const std::bad_alloc &) {
    return CDSGD_ERR_DEVICE;
}


int cdsgd_plan_set_thresholds(cdsgd_plan *plan, const float *thresholds)
try {
    if (!plan) return CDSGD_ERR_NULL;
    bool all_pow2 = true, any_tiny = false;
    if (thresholds)
        for (int i = 0; i < plan->num_tensors; ++i) {
            if (!good_threshold(thresholds[i])) return CDSGD_ERR_PARAM;
            all_pow2 = all_pow2 && is_pow2_threshold(thresholds[i]);
            any_tiny = any_tiny || is_tiny_threshold(thresholds[i]);
        }
    std::vector<TensorDesc> next = plan->host_tensors;
    for (int i = 0; i < plan->num_tensors; ++i) next[(size_t)i].threshold = thresholds ? thresholds[i] : 0.0f;
    if (hipMemcpy(plan->tensors, next.data(), sizeof(TensorDesc) * next.size(), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        return CDSGD_ERR_DEVICE;
    }
    plan->host_tensors.swap(next);
    plan->own_thresholds = thresholds != nullptr;
    plan->own_thresholds_pow2 = thresholds != nullptr && all_pow2;
    plan->own_thresholds_tiny = any_tiny;
    return CDSGD_OK;
} catch (const std::bad_alloc &) {
    return CDSGD_ERR_DEVICE;
}

size_t cdsgd_sparse_segments(size_t n) { return ((n + 15) / 16 + kSegWords - 1) / kSegWords; }

size_t cdsgd_sparse_words(size_t n) { return cdsgd_sparse_segments(n) * kSegStride; }

int cdsgd_sparse_encode(const uint32_t *packed, size_t n, uint32_t *sparse, uint32_t *segment_words,
                        void *hip_stream)
{
    if (!packed || !sparse) return CDSGD_ERR_NULL;
    if (n == 0 || cdsgd_sparse_segments(n) > kMaxGrid) return CDSGD_ERR_SIZE;
    if (!aligned(packed, 4) || !aligned(sparse, 4) || !aligned(segment_words, 4)) return CDSGD_ERR_ALIGN;
    const size_t pb = (size_t)packed_bytes_of(n), sb = cdsgd_sparse_words(n) * 4, cb = cdsgd_sparse_segments(n) * 4;
    if (overlap2(packed, pb, sparse, sb) || overlap2(packed, pb, segment_words, cb) ||
        overlap2(sparse, sb, segment_words, cb))
        return CDSGD_ERR_ALIAS;
    const unsigned segments = (unsigned)cdsgd_sparse_segments(n);
    hipLaunchKernelGGL(k_sparse_encode, dim3((segments + kEncodeWaves - 1u) / kEncodeWaves), dim3(64 * kEncodeWaves), 0,
                       (hipStream_t)hip_stream, packed, (unsigned long long)((n + 15) / 16), sparse, segment_words, segments);
    return launch_status();
}

int cdsgd_decode_sum_sparse(const uint32_t *const *sparse, int num_workers, float *agg, size_t n, float threshold,
                            void *hip_stream)
{
    if (!sparse || !agg) return CDSGD_ERR_NULL;
    if (n == 0 || chunks_of(n) > kMaxGrid) return CDSGD_ERR_SIZE;
    if (!good_threshold(threshold)) return CDSGD_ERR_PARAM;
    if (num_workers < 1 || num_workers > CDSGD_MAX_WORKERS) return CDSGD_ERR_WORKERS;
    for (int j = 0; j < num_workers; ++j)
        if (!sparse[j]) return CDSGD_ERR_NULL;
    if (!aligned(agg, 16)) return CDSGD_ERR_ALIGN;
    for (int j = 0; j < num_workers; ++j)
        if (!aligned(sparse[j], 4)) return CDSGD_ERR_ALIGN;
    for (int j = 0; j < num_workers; ++j)
        if (overlap2(sparse[j], cdsgd_sparse_words(n) * 4, agg, n * sizeof(float))) return CDSGD_ERR_ALIAS;
    return launch_decode_sum<true>(sparse, num_workers, agg, n, threshold, hip_stream);
}

int cdsgd_plan_set_peer_format(cdsgd_plan *plan, int format)
{
    if (!plan) return CDSGD_ERR_NULL;
    if (format != CDSGD_PEERS_PACKED && format != CDSGD_PEERS_SPARSE) return CDSGD_ERR_PARAM;
    plan->peers_sparse = format == CDSGD_PEERS_SPARSE;
    return CDSGD_OK;
}

int cdsgd_probe_streams(const float *const *reads, int num_reads, float *const *writes, int num_writes, size_t n,
                        float *sink, unsigned lds_bytes, void *hip_stream)
{
    if (num_reads < 0 || num_reads > kProbeMaxReads || num_writes < 0 || num_writes > kProbeMaxWrites ||
        num_reads + num_writes == 0 || lds_bytes > 65536u)
        return CDSGD_ERR_PARAM;
    if ((num_reads > 0 && !reads) || (num_writes > 0 && !writes) || (num_writes == 0 && !sink)) return CDSGD_ERR_NULL;
    if (n == 0 || n % 256 != 0 || n / 256 > 0xFFFFFFFFull / 64) return CDSGD_ERR_SIZE;
    ProbeStreams p;
    std::memset(&p, 0, sizeof(p));
    p.num_reads = num_reads;
    for (int i = 0; i < num_reads; ++i) {
        if (!reads[i]) return CDSGD_ERR_NULL;
        if (!aligned(reads[i], 16)) return CDSGD_ERR_ALIGN;
        p.r[i] = reads[i];
    }
    for (int i = 0; i < num_writes; ++i) {
        if (!writes[i]) return CDSGD_ERR_NULL;
        if (!aligned(writes[i], 16)) return CDSGD_ERR_ALIGN;
        for (int j = 0; j < num_reads; ++j)
            if (overlap(writes[i], reads[j], n * sizeof(float))) return CDSGD_ERR_ALIAS;
        for (int j = 0; j < i; ++j)
            if (overlap(writes[i], writes[j], n * sizeof(float))) return CDSGD_ERR_ALIAS;
        p.w[i] = writes[i];
    }
    const dim3 grid((unsigned)(n / 256)), block(64);
    hipStream_t s = (hipStream_t)hip_stream;
#define CDSGD_PROBE(R, W) hipLaunchKernelGGL((k_probe_streams<R, W>), grid, block, lds_bytes, s, p, sink)
    switch ((num_reads > 3 ? 4 : num_reads) * 4 + num_writes) {
    case 4 * 4 + 0: CDSGD_PROBE(-1, 0); break;
    case 4 * 4 + 1: CDSGD_PROBE(-1, 1); break;
    case 4 * 4 + 2: CDSGD_PROBE(-1, 2); break;
    case 4 * 4 + 3: CDSGD_PROBE(-1, 3); break;
    case 0 * 4 + 1: CDSGD_PROBE(0, 1); break;
    case 0 * 4 + 2: CDSGD_PROBE(0, 2); break;
    case 0 * 4 + 3: CDSGD_PROBE(0, 3); break;
    case 1 * 4 + 0: CDSGD_PROBE(1, 0); break;
    case 1 * 4 + 1: CDSGD_PROBE(1, 1); break;
    case 1 * 4 + 2: CDSGD_PROBE(1, 2); break;
    case 1 * 4 + 3: CDSGD_PROBE(1, 3); break;
    case 2 * 4 + 0: CDSGD_PROBE(2, 0); break;
    case 2 * 4 + 1: CDSGD_PROBE(2, 1); break;
    case 2 * 4 + 2: CDSGD_PROBE(2, 2); break;
    case 2 * 4 + 3: CDSGD_PROBE(2, 3); break;
    case 3 * 4 + 0: CDSGD_PROBE(3, 0); break;
    case 3 * 4 + 1: CDSGD_PROBE(3, 1); break;
    case 3 * 4 + 2: CDSGD_PROBE(3, 2); break;
    default: CDSGD_PROBE(3, 3); break;
    }
#undef CDSGD_PROBE
    return launch_status();
}

int cdsgd_plan_set_max_workgroups(cdsgd_plan *plan, int max_workgroups)
{
    if (!plan) return CDSGD_ERR_NULL;
    if (max_workgroups < 0) return CDSGD_ERR_PARAM;
    plan->max_workgroups = (unsigned)max_workgroups;
    return CDSGD_OK;
}

int cdsgd_step_warmup(cdsgd_plan *plan, long i, long warmup_steps, float lr_local, float lr_global,
                      void *hip_stream)
{
    if (!plan) return CDSGD_ERR_NULL;
    if (warmup_steps < 0 || i < 0 || i > warmup_steps || !std::isfinite(lr_local) || !std::isfinite(lr_global))
        return CDSGD_ERR_PARAM;
    const int mode = i == warmup_steps ? kLocalRule : (i == warmup_steps - 1 ? kLocalCopy : kLocalNone);
    return launch_full_pass(plan, mode, lr_local, lr_global, hip_stream);
}

int cdsgd_trainer_create(cdsgd_plan *plan, long warmup_steps, int k, float threshold, float lr_local,
                         float lr_global, cdsgd_trainer **out)
{
    if (!out) return CDSGD_ERR_NULL;
    *out = nullptr;
    if (!plan) return CDSGD_ERR_NULL;
    if (warmup_steps < 0 || k < 1 || !good_threshold(threshold) || !std::isfinite(lr_local) ||
        !std::isfinite(lr_global))
        return CDSGD_ERR_PARAM;
    cdsgd_trainer *t = new (std::nothrow) cdsgd_trainer;
    if (!t) return CDSGD_ERR_DEVICE;
    t->plan = plan;
    t->warmup_steps = warmup_steps;
    t->k = k;
    t->threshold = threshold;
    t->lr_local = lr_local;
    t->lr_global = lr_global;
    t->iteration = 0;
    *out = t;
    return CDSGD_OK;
}

int cdsgd_trainer_step(cdsgd_trainer *trainer, void *hip_stream, int *pass_kind)
{
    if (!trainer) return CDSGD_ERR_NULL;
    const long it = trainer->iteration;
    int rc, kind;
    if (it <= trainer->warmup_steps) {
        kind = CDSGD_PASS_WARMUP;
        rc = cdsgd_step_warmup(trainer->plan, it, trainer->warmup_steps, trainer->lr_local, trainer->lr_global,
                               hip_stream);
    } else {
        const long count = it - trainer->warmup_steps - 1;
        kind = (count % trainer->k) != 0 ? CDSGD_PASS_COMPRESSED : CDSGD_PASS_CORRECTION;
        rc = cdsgd_step_fused(trainer->plan, count, trainer->k, trainer->threshold, trainer->lr_local,
                              trainer->lr_global, hip_stream);
    }
    if (rc != CDSGD_OK) return rc;  // the iteration counter only advances on success
    trainer->iteration = it + 1;
    if (pass_kind) *pass_kind = kind;
    return CDSGD_OK;
}

long cdsgd_trainer_iteration(const cdsgd_trainer *trainer) { return trainer ? trainer->iteration : -1; }

int cdsgd_trainer_destroy(cdsgd_trainer *trainer)
{
    delete trainer;
    return CDSGD_OK;
}

}  // extern "C"

namespace {

std::mutex g_static_mutex;
constexpr int kStaticMaxDevices = 64;
unsigned char *g_static_ptr[kStaticMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device.
int static_scratch(unsigned char **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kStaticMaxDevices) {
        (void)hipGetLastError();
        return CDSGD_ERR_DEVICE;
    }
    std::lock_guard<std::mutex> lock(g_static_mutex);
    if (!g_static_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return CDSGD_ERR_DEVICE;
        }
        g_static_ptr[dev] = static_cast<unsigned char *>(p);
    }
    *out = g_static_ptr[dev];
    return CDSGD_OK;
}

template <typename Payload>
int launch_static_build(const StaticTarget &to, const Payload &p, hipStream_t s)
{
    const unsigned work = to.slots > to.count * to.row ? to.slots : to.count * to.row;
    const unsigned blocks = (work + 255u) / 256u;
    hipLaunchKernelGGL((k_static_build<Payload>), dim3(blocks < 1024u ? blocks : 1024u), dim3(256), 0, s, to, p);
    return launch_status();
}

// Tensor 0's buffers, and its stream of each of the first `streams` workers; no tensors yet.
void arenas_of(const cdsgd_tensor *tensors, const uint32_t *const *const *peers, int streams, int self, StaticArenas *flat)
{
    std::memset(flat, 0, sizeof(*flat));
    const cdsgd_tensor &z = tensors[0];
    const void *const role[kStaticRoles] = {z.w_global, z.w_local, z.residual, z.grad, z.packed_self, z.agg_full};
    for (int r = 0; r < kStaticRoles; ++r) flat->role[r] = (unsigned long long)reinterpret_cast<uintptr_t>(role[r]);
    for (int j = 0; j < streams; ++j)
        if (j != self) flat->stream[j] = reinterpret_cast<const uint8_t *>(peers[j][0]);
}

// The compressed pass over a checked list in arenas of at most StaticArenas::kTensors tensors, described by the launch's
// own arguments; `shape` has kArena.
int launch_from_arguments(const cdsgd_tensor *tensors, int num_tensors, const uint32_t *const *const *peers, int num_workers,
                          int self, int grad_dtype, const unsigned *offsets, unsigned num_chunks,
                          const CompressedLaunch &shape, int form, float threshold, float lr_local, float lr_global, hipStream_t s)
{
    StaticArenas flat;
    arenas_of(tensors, peers, num_workers, self, &flat);
    unsigned slots = 0;
    for (unsigned k = 0; k < StaticArenas::kTensors; ++k) {
        if (k >= (unsigned)num_tensors) {
            flat.slots[k] = StaticArenas::kNoSlot;
            continue;
        }
        flat.offsets[k] = offsets[k];
        flat.sizes[k] = (unsigned)tensors[k].n;
        flat.slots[k] = slots;
        slots += (unsigned)chunks_of(tensors[k].n);
    }
    const unsigned num_tiles = num_chunks * (kChunkQuads / (64u * shape.waves));
    const float scale = lr_global / (float)num_workers;
    const auto bound = [&](unsigned used) { return shape.lds <= used ? 0u : shape.lds - used; };
    // (17 to 32 workers ask for all streams at once, as the kernels with tables do not: weights behind gradient and residual over that,
    // 2.2 / 5 / 12 / 20 M: chain N = 17 .99 .99 1.00 1.01, 24 .99 .99 1.00 .99, 32 .98 1.00 1.00 .99, bf16 .98 .99 .99 .99;  count
    // N = 17 1.03 1.01 1.00 1.02, 20 1.02 1.01 1.01 1.03, 24 1.01 1.00 1.01 1.00, 32 1.00 1.00 .99 1.00.)
#define CDSGD_LAUNCH_ARGUMENTS_S(SZ, WAVES, FORM, GT, HOW)                                                     \
    hipLaunchKernelGGL((k_fused_arguments<SZ, WAVES, FORM, GT, HOW>), dim3(num_tiles), dim3(64 * WAVES),       \
                       bound(kTileLds<SZ, FORM, WAVES, false, true>), s, num_tiles, (unsigned)num_tensors, num_workers, self, threshold, \
                       lr_local, scale, flat)
#define CDSGD_LAUNCH_ARGUMENTS(SZ, WAVES, FORM, HOW)                                                           \
    do {                                                                                                       \
        if (grad_dtype == CDSGD_GRAD_BF16) CDSGD_LAUNCH_ARGUMENTS_S(SZ, WAVES, FORM, kGradBF16, HOW);          \
        else if (grad_dtype == CDSGD_GRAD_F16) CDSGD_LAUNCH_ARGUMENTS_S(SZ, WAVES, FORM, kGradF16, HOW);       \
        else CDSGD_LAUNCH_ARGUMENTS_S(SZ, WAVES, FORM, kGradF32, HOW);                                         \
    } while (0)
#define CDSGD_LAUNCH_ARGUMENTS_32BIT(SZ, WAVES, FORM, HOW)                                                     \
    do {                                                                                                       \
        if (grad_dtype != CDSGD_GRAD_F32) return CDSGD_ERR_DEVICE;                                             \
        CDSGD_LAUNCH_ARGUMENTS_S(SZ, WAVES, FORM, kGradF32, HOW);                                              \
    } while (0)
#define CDSGD_LAUNCH_ARGUMENTS_F(FORM, LAUNCH_LATE)                                                            \
    do {                                                                                                       \
        if (shape.waves == 1u) CDSGD_LAUNCH_ARGUMENTS(kUpTo8, 1, FORM, kArena);                                \
        else if (num_workers <= kUpTo8) CDSGD_LAUNCH_ARGUMENTS(kUpTo8, 4, FORM, kArena);                       \
        else if (num_workers > kUpTo32) CDSGD_LAUNCH_ARGUMENTS(kAnyWorkers, 4, FORM, kArena);                  \
        else if (num_workers > kUpTo16 && (shape.how & kWrittenOut)) CDSGD_LAUNCH_ARGUMENTS(kUpTo32, 4, FORM, kWrittenOut | kArena); \
        else if (num_workers > kUpTo16) CDSGD_LAUNCH_ARGUMENTS(kUpTo32, 4, FORM, kArena);                      \
        else if (shape.how & kLate) LAUNCH_LATE(kUpTo16, 4, FORM, kWrittenOut | kLate | kArena);               \
        else if (shape.how & kWrittenOut) CDSGD_LAUNCH_ARGUMENTS(kUpTo16, 4, FORM, kWrittenOut | kArena);      \
        else CDSGD_LAUNCH_ARGUMENTS(kUpTo16, 4, FORM, kArena);                                                 \
    } while (0)
    if (form == kCount) CDSGD_LAUNCH_ARGUMENTS_F(kCount, CDSGD_LAUNCH_ARGUMENTS_32BIT);
    else CDSGD_LAUNCH_ARGUMENTS_F(kChain, CDSGD_LAUNCH_ARGUMENTS);
#undef CDSGD_LAUNCH_ARGUMENTS_F
#undef CDSGD_LAUNCH_ARGUMENTS_32BIT
#undef CDSGD_LAUNCH_ARGUMENTS
#undef CDSGD_LAUNCH_ARGUMENTS_S
    return launch_status();
}

// Write the tables of a checked layer list into the static array at `base`.
// offsets: of a list in arenas (in_arenas), or null; arena_chunks: the chunk table holds ArenaChunk entries (lists in arenas only).
int build_static_tables(unsigned char *base, const cdsgd_tensor *tensors, int num_tensors,
                        const uint32_t *const *const *peers, int num_workers, int self, int grad_dtype, bool with_rows,
                        const unsigned *offsets, bool arena_chunks, hipStream_t s)
{
    const bool arenas = offsets != nullptr;
    const unsigned grad_bytes = grad_dtype == CDSGD_GRAD_F32 ? 4u : 2u;
    StaticTarget to;
    to.desc = reinterpret_cast<TensorDesc *>(base + kStaticOffDesc);
    to.chunks = reinterpret_cast<ChunkRef *>(base + kStaticOffChunks);
    to.rows = reinterpret_cast<const uint8_t **>(base + kStaticOffPeers);
    to.arena_chunks = arena_chunks ? reinterpret_cast<ArenaChunk *>(base + kStaticOffChunks) : nullptr;
    to.row = with_rows ? row_entries(num_workers) : 0u;
    to.workers = with_rows ? (unsigned)num_workers : 0u;
    to.self = (unsigned)self;
    to.grad_bytes = grad_bytes;
    to.slot0 = 0;
    const int streams = (int)to.workers;
    const auto bits = [](const void *p) { return (unsigned long long)reinterpret_cast<uintptr_t>(p); };
    StaticArenas flat;
    StaticPointers any;
    if (arenas) arenas_of(tensors, peers, streams, self, &flat);
    else std::memset(&any, 0, sizeof(any));
    const unsigned stride = StaticPointers::stride(to.workers);
    const unsigned part = arenas ? StaticArenas::kTensors : StaticPointers::kWords / stride;
    for (int first = 0; first < num_tensors; first += (int)part) {
        const unsigned left = (unsigned)(num_tensors - first);
        to.first = (unsigned)first;
        to.count = left < part ? left : part;
        to.slots = 0;
        for (unsigned k = 0; k < to.count; ++k) {
            const int i = first + (int)k;
            const cdsgd_tensor &t = tensors[i];
            if (arenas) {
                flat.offsets[k] = offsets[i];
                flat.sizes[k] = (unsigned)t.n;
                flat.slots[k] = to.slots;
            } else {
                unsigned long long *w = any.w + (size_t)k * stride;
                const void *const role[kStaticRoles] = {t.w_global, t.w_local, t.residual, t.grad, t.packed_self, t.agg_full};
                *w++ = (unsigned long long)t.n | (unsigned long long)to.slots << 32;
                for (int r = 0; r < kStaticRoles; ++r) *w++ = bits(role[r]);
                for (int j = 0; j < streams; ++j) *w++ = j == self ? 0ull : bits(peers[j][i]);
            }
            to.slots += (unsigned)chunks_of(t.n);
        }
        const int rc = arenas ? launch_static_build(to, flat, s) : launch_static_build(to, any, s);
        if (rc != CDSGD_OK) return rc;
        to.slot0 += to.slots;
    }
    return CDSGD_OK;
}

}  // namespace

extern "C" int cdsgd_step_fused_static(const cdsgd_tensor *tensors, int num_tensors,
                                       const uint32_t *const *const *peers, int num_workers, int self,
                                       int grad_dtype, long step, int k, float threshold, float lr_local,
                                       float lr_global, void *hip_stream)
{
    unsigned long long total_chunks = 0;
    bool all_agg = true;
    int rc = check_layer_list(tensors, num_tensors, peers, num_workers, self, grad_dtype, &total_chunks, &all_agg);
    if (rc != CDSGD_OK) return rc;
    if (!good_step_params(step, k, threshold, lr_local, lr_global)) return CDSGD_ERR_PARAM;
    if (num_tensors > kStaticMaxTensors || total_chunks > kStaticMaxChunks) return CDSGD_ERR_SIZE;
    const bool compressed = (step % k) != 0;
    if (!compressed && num_workers > 1 && !all_agg) return CDSGD_ERR_NULL;

    unsigned char *base = nullptr;
    rc = static_scratch(&base);
    if (rc != CDSGD_OK) return rc;
    hipStream_t s = (hipStream_t)hip_stream;

    PlanTables pt;
    pt.tensors = reinterpret_cast<TensorDesc *>(base + kStaticOffDesc);
    pt.chunks = reinterpret_cast<ChunkRef *>(base + kStaticOffChunks);
    pt.rows = reinterpret_cast<const uint8_t **>(base + kStaticOffPeers);
    pt.num_tensors = num_tensors;
    pt.num_workers = num_workers;
    pt.self = self;
    pt.num_chunks = (unsigned)total_chunks;
    pt.has_agg_full = all_agg;
    pt.grad_type = grad_dtype;

    unsigned offsets[kStaticMaxTensors];
    const bool arenas = in_arenas(tensors, num_tensors, peers, compressed ? num_workers : 0, self,
                                  grad_dtype == CDSGD_GRAD_F32 ? 4u : 2u, offsets);
    if (compressed && arenas) {
        pt.arena_chunks = reinterpret_cast<ArenaChunk *>(base + kStaticOffChunks);
        int form;
        CompressedLaunch shape = launch_of_pass(&pt, threshold, &form);
        const bool chunks = (shape.how & kArena) != 0;
        // (above 32 workers the kernel for arenas is the slower one, by less than the launch that it spares)
        if (shape.how == 0 && num_workers > kUpTo32 && form != kChainTiny && total_chunks * kTilesPerChunk <= kMidListTiles)
            shape.how = kArena;
        if ((shape.how & kArena) != 0 && num_tensors <= (int)StaticArenas::kTensors)
            return launch_from_arguments(tensors, num_tensors, peers, num_workers, self, grad_dtype, offsets, (unsigned)total_chunks,
                                         shape, form, threshold, lr_local, lr_global, s);
        if (!chunks) pt.arena_chunks = nullptr;
    }
    rc = build_static_tables(base, tensors, num_tensors, peers, num_workers, self, grad_dtype, compressed, arenas ? offsets : nullptr,
                             pt.arena_chunks != nullptr, s);
    if (rc != CDSGD_OK) return rc;
    return launch_formal_pass(&pt, step, k, threshold, lr_local, lr_global, true, hip_stream);
}
