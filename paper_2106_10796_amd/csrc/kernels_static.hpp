// Tables built on the device for the entry point that allocates nothing, and their layout.
#pragma once

namespace {

// ---------------------------------------------------------------------------
// tables built on the device, for the entry point that allocates nothing
// ---------------------------------------------------------------------------
// The layer list travels in the arguments of one or more launches of k_static_build, each of which writes the
// descriptors, the rows of stream pointers and the chunk table entries of the tensors it carries.  Bound by launches
// (2-4 us each) and nothing else, so what matters is how many tensors fit the 4 KiB that a kernel's arguments may
// take.  Lists whose buffers lie in arenas, every buffer of tensor i at the same element offset from tensor 0's (what
// a program with flat gradient buckets has), need an offset per tensor: 256 tensors a launch.  Any other list needs
// its pointers: 464 / (7 + workers) tensors a launch.  (ResNet-50-shaped list, N = 8, fp16 gradients: 9 launches of
// 3 KiB of finished tables and one for the chunk table took 22 us of the call's 113; one launch takes 4.5 of 100.)
constexpr int kStaticRoles = 6;  // w_global, w_local, residual, grad, packed_self, agg_full

struct StaticTarget {
    TensorDesc *desc;
    ChunkRef *chunks;
    ArenaChunk *arena_chunks;  // in place of `chunks`, or null
    const uint8_t **rows;
    unsigned first, count;   // tensors [first, first + count) of the list
    unsigned slot0, slots;   // their entries of the chunk table
    unsigned row;            // entries of a row of stream pointers; 0: the pass reads none
    unsigned workers, self, grad_bytes;
};

struct StaticArenas {
    static constexpr unsigned kTensors = 256;
    unsigned long long role[kStaticRoles];            // tensor 0's buffers (0: none)
    const uint8_t *stream[CDSGD_MAX_WORKERS];         // tensor 0's stream of every worker (null: the own, and past the last)
    // per tensor: first chunk table entry (counted from slot0; kNoSlot past the last), offset in 16 elements, elements
    __attribute__((aligned(16))) unsigned slots[kTensors];
    unsigned offsets[kTensors], sizes[kTensors];
    static constexpr unsigned kNoSlot = 0xFFFFFFFFu;

    __device__ unsigned n(unsigned i, unsigned) const { return sizes[i]; }
    __device__ unsigned slot(unsigned i, unsigned) const { return slots[i]; }
    __device__ unsigned off16(unsigned i) const { return offsets[i]; }
    __device__ unsigned long long buffer(unsigned i, int r, unsigned grad_bytes, unsigned) const
    {
        if (role[r] == 0ull) return 0ull;
        const unsigned long long off = (unsigned long long)offsets[i];
        return role[r] + (r == 4 ? off * 4u : off * 16u * (r == 3 ? grad_bytes : 4u));
    }
    __device__ unsigned long long of_worker(unsigned i, unsigned j, unsigned) const
    {
        return reinterpret_cast<unsigned long long>(stream[j]) + (unsigned long long)offsets[i] * 4u;
    }
};

struct StaticPointers {
    static constexpr unsigned kWords = 464;
    // per tensor: elements and first chunk table entry, the buffers, the workers' streams
    unsigned long long w[kWords];

    __device__ __host__ static constexpr unsigned stride(unsigned workers) { return 1u + kStaticRoles + workers; }
    __device__ unsigned n(unsigned i, unsigned workers) const { return (unsigned)w[i * stride(workers)]; }
    __device__ unsigned slot(unsigned i, unsigned workers) const { return (unsigned)(w[i * stride(workers)] >> 32); }
    __device__ unsigned off16(unsigned) const { return 0u; }  // (lists in arenas only)
    __device__ unsigned long long buffer(unsigned i, int r, unsigned, unsigned workers) const
    {
        return w[i * stride(workers) + 1u + (unsigned)r];
    }
    __device__ unsigned long long of_worker(unsigned i, unsigned j, unsigned workers) const
    {
        return w[i * stride(workers) + 1u + kStaticRoles + j];
    }
};

constexpr unsigned kStaticMaxPart = StaticArenas::kTensors;  // most tensors of one launch

template <typename Payload>
__global__ __launch_bounds__(256) void k_static_build(StaticTarget to, Payload p)
{
    __shared__ unsigned starts[kStaticMaxPart];
    for (unsigned i = threadIdx.x; i < to.count; i += 256u) starts[i] = p.slot(i, to.workers);
    __syncthreads();
    const unsigned id = blockIdx.x * 256u + threadIdx.x, step = gridDim.x * 256u;
    for (unsigned i = id; i < to.count; i += step) {
        const unsigned n = p.n(i, to.workers);
        TensorDesc d;
        d.w_global = reinterpret_cast<float *>(p.buffer(i, 0, to.grad_bytes, to.workers));
        d.w_local = reinterpret_cast<float *>(p.buffer(i, 1, to.grad_bytes, to.workers));
        d.residual = reinterpret_cast<float *>(p.buffer(i, 2, to.grad_bytes, to.workers));
        d.grad = reinterpret_cast<const void *>(p.buffer(i, 3, to.grad_bytes, to.workers));
        d.packed_self = reinterpret_cast<uint8_t *>(p.buffer(i, 4, to.grad_bytes, to.workers));
        d.agg_full = reinterpret_cast<const float *>(p.buffer(i, 5, to.grad_bytes, to.workers));
        d.ext.full_chunks = n / kChunkElems;
        d.ext.tail_elems = n % kChunkElems;
        d.ext.tail_bytes = (d.ext.tail_elems + 15u) / 16u * 4u;
        d.ext.pad_ = 0u;
        d.threshold = 0.0f;
        d.pad_ = 0u;
        to.desc[to.first + i] = d;
    }
    for (unsigned e = id; e < to.count * to.row; e += step) {
        const unsigned i = e / to.row, j = e % to.row;
        to.rows[to.first * to.row + e] =
            j < to.workers && j != to.self ? reinterpret_cast<const uint8_t *>(p.of_worker(i, j, to.workers)) : nullptr;
    }
    for (unsigned s = id; s < to.slots; s += step) {
        unsigned lo = 0, hi = to.count;  // invariant: starts[lo] <= s < starts[hi] (the total behind the last one)
        while (hi - lo > 1) {
            const unsigned mid = (lo + hi) >> 1;
            if (starts[mid] <= s) lo = mid;
            else hi = mid;
        }
        const unsigned chunk = s - starts[lo];
        if (to.arena_chunks) {
            const unsigned left = p.n(lo, to.workers) - chunk * kChunkElems;
            ArenaChunk at;
            at.off16 = p.off16(lo) + chunk * (kChunkElems / 16u);
            at.elems = left < kChunkElems ? left : kChunkElems;
            to.arena_chunks[to.slot0 + s] = at;
        } else {
            ChunkRef cr;
            cr.tensor = to.first + lo;
            cr.chunk = chunk;
            to.chunks[to.slot0 + s] = cr;
        }
    }
}

// The compressed pass over a list in arenas that fits one launch's arguments: no tables, one launch instead of two.  A wave
// finds the tensor of its chunk by comparing the chunk's number with the first chunks of all of them, four to a lane, and
// the chunk's place in the arenas follows from the tensor's entry: two trips to memory in front of the data, as with tables.
// Bound by HBM above some million elements and by the launch below.  Time of the call, tables first / now, us: 10 k to 300 k
// elements, N = 2 to 32 8.4 / 4.9, 1 M, N = 8, fp16 9.3 / 6.3, 4 M, N = 16 22.3 / 19.2, 14 M, N = 16, bf16 57.5 / 54.4;
// ResNet-20-shaped, N = 8 10.0 / 6.6; ResNet-50-shaped, N = 2 101.3 / 100.5, N = 8, fp16 95.2 / 93.5, N = 16, bf16 104.3 /
// 100.8; above 16 workers 1 M, N = 32 10.8 / 7.0, 4 M, N = 64 31.5 / 28.5.
template <int SZ, int WAVES, int FORM, int GT, int HOW>
__global__ __launch_bounds__(64 * WAVES) void k_fused_arguments(unsigned num_tiles, unsigned num_tensors, int num_workers, int self,
                                                                float t, float lr_local, float scale, StaticArenas p)
{
    static_assert((HOW & kArena) != 0, "lists in arenas");
    __shared__ __attribute__((aligned(16))) uint8_t lds[kTileLds<SZ, FORM, WAVES, false, true>];
    constexpr unsigned kQuads = 64u * WAVES, kPerChunk = kChunkQuads / kQuads;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    admit_six_groups<SZ, FORM, HOW & ~kArena>();
    const unsigned lane = threadIdx.x & 63u;
    const unsigned x = piece_of_workgroup<true>((unsigned)blockIdx.x, kPerChunk, num_tiles);
    const unsigned slot = x / kPerChunk, tile = x % kPerChunk;
    StreamPointers<SZ, WAVES, false> from;
    from.template load<false>(p.stream, num_workers, wave, lane);
    TensorDesc d;
    d.w_global = reinterpret_cast<float *>(p.role[0]);
    d.w_local = reinterpret_cast<float *>(p.role[1]);
    d.residual = reinterpret_cast<float *>(p.role[2]);
    d.grad = reinterpret_cast<const void *>(p.role[3]);
    d.packed_self = reinterpret_cast<uint8_t *>(p.role[4]);
    from.pin();
    unsigned i = 0;
    if (num_tensors > 1u) {
        static_assert(StaticArenas::kTensors == 256, "four tensors to a lane");
        const u4 first = *reinterpret_cast<const u4 *>(p.slots + 4u * lane);
        unsigned begun = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) begun += (unsigned)__builtin_popcountll(__ballot(first[c] <= slot));
        i = begun - 1u;
    }
    const unsigned chunk = slot - p.slots[i], left = p.sizes[i] - chunk * kChunkElems;
    const unsigned elems = left < kChunkElems ? left : kChunkElems;
    const unsigned quad = (p.offsets[i] + chunk * (kChunkElems / 16u)) * 4u, bytes = (elems + 15u) / 16u * 4u;
    d.ext.full_chunks = 0u;
    d.ext.tail_bytes = quad + bytes;  // where the chunk's codes end in a stream
    if (elems == kChunkElems) {
        fused_tile<false, SZ, WAVES, FORM, GT, false, HOW, false, false>(d, from, num_workers, self, quad, tile, kQuads * 4u, kQuads, t, lr_local,
                                                           scale, true, lds);
    } else if (tile * kQuads < bytes) {
        const unsigned elems0 = tile * kQuads * 4u;
        fused_tile<true, SZ, WAVES, FORM, GT, false, HOW, false, false>(d, from, num_workers, self, quad, tile, elems_from(elems0, elems),
                                                          bytes - tile * kQuads, t, lr_local, scale, true, lds);
    }
}

static_assert(sizeof(StaticTarget) + sizeof(StaticArenas) <= 3840 && sizeof(StaticTarget) + sizeof(StaticPointers) <= 3840,
              "4 KiB of arguments, 256 bytes of which the runtime fills in");

// Layout of the static device array: descriptor table, rows of stream pointers, chunk table; every
// region starts on a 256-byte boundary.
constexpr size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr int kStaticMaxTensors = CDSGD_STATIC_MAX_TENSORS;
constexpr unsigned kStaticMaxChunks = CDSGD_STATIC_MAX_CHUNKS;
constexpr size_t kStaticOffDesc = 0;
constexpr size_t kStaticOffPeers = round256(sizeof(TensorDesc) * kStaticMaxTensors);
constexpr size_t kStaticOffChunks =
    round256(kStaticOffPeers + sizeof(void *) * ((size_t)kStaticMaxTensors * row_entries(CDSGD_MAX_WORKERS) + CDSGD_MAX_WORKERS));
constexpr size_t kStaticBytes = kStaticOffChunks + sizeof(ChunkRef) * (size_t)kStaticMaxChunks;
static_assert(kChunkElems == CDSGD_STATIC_CHUNK_ELEMS, "the header states the chunk size the limit is counted in");

}  // namespace
