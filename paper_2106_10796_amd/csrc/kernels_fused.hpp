// Kernels over a layer list: the fused compressed pass (a1-a6) and the passes on 32-bit gradients.
#pragma once

namespace {

// ---------------------------------------------------------------------------
// Fused compressed step (a1-a6), one group of waves per tile of a chunk
// ---------------------------------------------------------------------------
// Bound by HBM (24 + N / 4 bytes per element): every load of a group is in flight at once, so a group's life is the
// table lookups (chunk, then descriptor and stream pointers together), one round trip to memory, the decode and the
// stores.  (Stream pointers fetched behind the descriptor, one worker after the other above 16 workers: layer ranges of
// a million elements, N = 16 169.3 us for 19 launches, 166.5 now; 300 k elements, N = 64 6.3 us, 6.1; 1 M elements
// decoded and updated, N = 64 29.6 us, 28.6.  Longer lists are bound by HBM and gain nothing.)
// A persistent grid whose groups fetch the next tile before they finish one is 15 % slower: its groups drift apart,
// and the streams' requests in flight with them (2^26 elements, N = 16: 0.366 ms against 0.293).
// Whether the local weights, which do not wait for the sums, are stored before the decode or beside the global ones:
// before, where the decode is long enough to hide the store and the list of workers short enough for it to matter
// (1 GiB buckets, t = 0.05, N = 16: 1.161 ms against 1.25; count form 1.194 against 1.150 at their best residencies).
template <int SZ, int FORM>
constexpr bool kLocalFirst = SZ == kUpTo16 && FORM != kCount;

// How a pass is compiled beside its sizes (compressed_launch says which and why).
//   kLate        the workers' words are asked for behind the tile's own streams instead of in front of them
//   kWrittenOut  results are written through the L2 of the compute die (kThroughStream)
//   kStreamWords the workers' words are read non-temporally
//   kArena       the list lies in arenas (ArenaChunk): entry, buffers and stream pointers come in one trip to memory
//   kSixGroups   no more than six groups to a compute unit
//   kFewGroups   few groups walk the list (compressed_launch): the count form asks for the words first, the chain form reads all rows at once
constexpr int kLate = 1, kWrittenOut = 2, kStreamWords = 4, kArena = 8, kSixGroups = 32, kFewGroups = 64;
template <int HOW>
struct ChunkEntry { typedef ChunkRef type; };
template <>
struct ChunkEntry<kArena> { typedef ArenaChunk type; };

// WAIT: the weights are asked for when gradient and residual are there, not with them: fewer streams in flight at a time, which
// memory serves a little faster in some passes (launch_formal_pass, with the times).
// MID: the chain's rows are written behind tests and its sums not spread over the banks (tile_put, tile_get).
template <bool G, int SZ, int WAVES, int FORM, int GT, bool SPARSE, int HOW, bool WAIT, bool MID>
__device__ __forceinline__ void fused_tile(const TensorDesc &d, const StreamPointers<SZ, WAVES, SPARSE> &from, int num_workers,
                                           int self, unsigned chunk, unsigned tile, unsigned rem_elems,
                                           unsigned rem_bytes, float t, float lr_local, float scale, bool write_local,
                                           uint8_t *lds)
{
    constexpr bool LATE = (HOW & kLate) != 0, OUT = (HOW & kWrittenOut) != 0, NT = (HOW & kStreamWords) != 0, FEW = (HOW & kFewGroups) != 0;
    constexpr int kStore = OUT ? kThroughStream : kStream;
    const unsigned tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane((int)(tid >> 6));
    // (kArena: `chunk` is the chunk's first quad, counted from tensor 0's)
    const size_t quad0 = (size_t)chunk * ((HOW & kArena) ? 1u : kChunkQuads) + tile * (64u * WAVES);
    const void *__restrict__ grad = grad_at<GT>(d.grad, quad0);
    float *__restrict__ resid = d.residual + 4 * quad0;
    float *__restrict__ wg = d.w_global + 4 * quad0;
    float *__restrict__ wl = d.w_local + 4 * quad0;
    uint8_t *pself = d.packed_self + quad0;

    TileStreams s;
    s.num_workers = num_workers;
    s.stream_bytes = d.ext.full_chunks * kChunkQuads + d.ext.tail_bytes;
    s.tile_at = (unsigned)quad0;
    s.segment_at = (size_t)chunk * (4u * kSegStride);
    s.tile = tile;
    unsigned words[kWordsPerWave<SZ>];
    if (!LATE) load_words<SZ, WAVES, SPARSE, NT>(words, from, s, wave, tid & 63u);
    if (FEW && FORM == kCount) __builtin_amdgcn_sched_barrier(0);
    const GradQuad<GT> loaded = load_grad<G, GT>(grad, tid, rem_elems);
    f4 r = ld4g<G>(resid, tid, rem_elems);
    f4 w;
    if (!WAIT) w = ld4g<G>(wg, tid, rem_elems);
    if (LATE) {
        __builtin_amdgcn_sched_barrier(0);
        load_words<SZ, WAVES, SPARSE, NT>(words, from, s, wave, tid & 63u);
    }

    // own codes: quantise, keep the residual, write what would be pushed
    const f4 g = widen<G, GT>(loaded, rem_elems);
    if (WAIT) {
        asm volatile("" ::"v"(g.x), "v"(r.x));
        __builtin_amdgcn_sched_barrier(0);
        w = ld4g<G>(wg, tid, rem_elems);
        __builtin_amdgcn_sched_barrier(0);
    }
    f4 sent;
    const unsigned own = quantize_quad(g, r, t, sent);
    st4g<G, kStore>(resid, tid, rem_elems, r);
    if (!G || tid < rem_bytes) st_code<OUT ? kThroughStream : 0>(pself, tid, own);

    // eq. 11 and eq. 10 from the same loaded weight
    f4 vl, vg;
#pragma unroll
    for (unsigned c = 0; c < 4; ++c) vl[c] = __builtin_fmaf(-lr_local, g[c], w[c]);
    if (kLocalFirst<SZ, FORM> && write_local) st4g<G, kStore>(wl, tid, rem_elems, vl);

    const f4 agg = tile_sums<SZ, FORM, WAVES, kSlotTests<SZ, SPARSE> || MID, !MID, FEW ? kAllFirst : 0>(words, own, sent, self, num_workers, t, lds);
#pragma unroll
    for (unsigned c = 0; c < 4; ++c) vg[c] = __builtin_fmaf(-scale, agg[c], w[c]);
    if (!kLocalFirst<SZ, FORM> && write_local) st4g<G, kStore>(wl, tid, rem_elems, vl);
    st4g<G, kStore>(wg, tid, rem_elems, vg);
}

// Lists in arenas, 17 to 32 workers: stream pointers and buffers are the same for every tile, and the compiler fetched them
// in front of the loop over tiles and kept them all through it: 4 to 18 of them in lanes of a vector register, and the
// chunk's entry asked for only behind the wait for them, one trip to memory more.  An offset that it cannot see through
// makes them the tile's own.  The kernels then need 81 to 92 scalar registers, which admit seven groups to a compute unit
// where 102 admit six, and long lists run better with six (kSix).  Time over that
// of the kernels before, so / with seven, N = 17 / 24 / 32:
//   t = 0.5, 32-bit   0.9 M .98 .99 .94 / .96 .98 .94;  1.5 M .98 .97 .97 / .98 .97 .97;  1.9 M .97 .97 .97 / .95 .95 .97;  3.5 to 26 M .99-1.00 / .99-1.00
//   t = 0.5, bf16     0.9 M .97 .98 .97 / .97 .98 .97;  1.5 M .99 .97 .99 / .99 .98 .99;  5 M .99 1.01 1.00 / 1.01 1.01 1.01;  12 and 16 M 1.00 / 1.01
//   t = 0.1, 32-bit   0.9 to 3.5 M .99-1.01 / .99-1.03;  12 and 16 M 1.00 / 1.01;  18 M .98 .99 1.00 / .97 .99 1.00
//   t = 0.1, bf16     0.9 M .99 .99 .96 / .99 .98 .96;  1.5 M .98 .97 .97;  3.5 M 1.00 .99 1.00;  12 and 16 M 1.00 / 1.01-1.02;  23 and 26 M .99-1.00 / .99-1.02
// (9 to 16 workers hold theirs through the loop in 98 to 106 registers and spill none; 93 to 101 before ragged ends were clipped.
// Time over that, N = 9 / 12 / 16: count form 32-bit 1.1 M 1.00 1.01 1.00, 1.6 M .99 .98 .98, 2.2 M 1.00 1.00 .98, 3 and 5 M .99-1.00,
// bf16 1.1 M .90 .93 .92, 1.6 M .91 .91 .89, 2.2 to 5 M .96-.99;  chain 0.3 and 0.5 M the launch, 1 to 12 M 32-bit .97-1.00, 0.9 and 1.6 M bf16 .94-.99.)
template <int SZ, int HOW>
constexpr bool kManyPointers = SZ == kUpTo32 && (HOW & kArena) != 0;

// Kernels of which a compute unit runs six groups (compressed_launch, with the times) although their registers would admit
// more: they name a scalar register that nothing uses.  A SIMD has 800; a wave takes its own and 16 more, in sixteens: 102
// admit six, 80 eight.  A bound by LDS takes as long and keeps 156 KiB of a compute unit's 160 from kernels of other streams.
template <int SZ, int FORM, int HOW>
constexpr bool kSix = kManyPointers<SZ, HOW> || (HOW & kSixGroups) != 0 || (SZ == kUpTo16 && FORM == kChain && (HOW & kLate) != 0);

template <int SZ, int FORM, int HOW>
__device__ __forceinline__ void admit_six_groups()
{
    if constexpr (kSix<SZ, FORM, HOW>) asm volatile("" ::: "s97");
}

// write_local: eq. 11 as well (false: the global half of a split step)
template <int SZ, int WAVES, int FORM, int GT, bool SPARSE, int HOW, bool WAIT>
__global__ __launch_bounds__(64 * WAVES) void k_fused_compressed(const TensorDesc *__restrict__ tensors,
                                                                 const typename ChunkEntry<HOW & kArena>::type *__restrict__ chunks,
                                                                 const uint8_t *const *__restrict__ rows,
                                                                 unsigned num_tiles, unsigned grid, int num_workers,
                                                                 int self, float t_call, float lr_local, float scale,
                                                                 int write_local)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[kTileLds<SZ, FORM, WAVES, SPARSE, true>];
    constexpr unsigned kQuads = 64u * WAVES, kPerChunk = kChunkQuads / kQuads;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // The kernels of 32-bit lists in arenas of 16 to 28 M elements, 17 to 32 workers: their groups are through sooner without the
    // tests and with the sums spread, and the order in which memory is asked is the worse one, at any residency.  Chain, time
    // over that so, 17 / 19 / 21 / 24 / 27 M elements: N = 17 1.02 1.03 1.02 1.01 1.00, 18 1.02 1.02 1.02 1.01 1.00, 20 1.02 1.01
    // 1.00 1.00 .99, 24 1.01 1.00 1.00 1.00 1.00, 28 and 32 1.00.  (16-bit gradients, N = 17, 18 M: even.)
    constexpr bool MID = kManyPointers<SZ, HOW> && (HOW & kWrittenOut) != 0 && !WAIT && GT == kGradF32;
    admit_six_groups<SZ, FORM, HOW>();
    for (unsigned b = blockIdx.x;;) {
        const unsigned x = piece_of_workgroup<true>(b, kPerChunk, num_tiles);
        const auto at = chunks[x / kPerChunk];
        const unsigned tile = x % kPerChunk;
        StreamPointers<SZ, WAVES, SPARSE> from;
        if constexpr ((HOW & kArena) != 0) {
            static_assert(!SPARSE, "arenas of packed streams");
            unsigned none = 0u;
            if constexpr (kManyPointers<SZ, HOW>) asm volatile("s_mov_b32 %0, 0" : "=s"(none));
            from.template load<false>(rows + none, num_workers, wave, threadIdx.x & 63u);
            TensorDesc d = tensors[none];
            from.pin();
            const unsigned quad = at.off16 * 4u, bytes = (at.elems + 15u) / 16u * 4u;
            d.ext.full_chunks = 0u;
            d.ext.tail_bytes = quad + bytes;  // where the chunk's codes end in a stream
            if (at.elems == kChunkElems) {
                fused_tile<false, SZ, WAVES, FORM, GT, SPARSE, HOW, WAIT, MID>(d, from, num_workers, self, quad, tile, kQuads * 4u, kQuads,
                                                                    t_call, lr_local, scale, write_local != 0, lds);
            } else if (tile * kQuads < bytes) {
                const unsigned elems0 = tile * kQuads * 4u;
                fused_tile<true, SZ, WAVES, FORM, GT, SPARSE, HOW, WAIT, MID>(d, from, num_workers, self, quad, tile,
                                                                   elems_from(elems0, at.elems), bytes - tile * kQuads,
                                                                   t_call, lr_local, scale, write_local != 0, lds);
            }
        } else {
            // (the select spares 9 to 16 sparse peers a load, 5-7 % of the time of the pass; up to 8 it costs long lists 1-2 %)
            from.template load<SZ == kUpTo16>(rows + (size_t)at.tensor * row_entries(num_workers), num_workers, wave, threadIdx.x & 63u);
            const TensorDesc d = tensors[at.tensor];
            from.pin();
            const float t = d.threshold > 0.0f ? d.threshold : t_call;
            if (at.chunk < d.ext.full_chunks) {
                fused_tile<false, SZ, WAVES, FORM, GT, SPARSE, HOW, WAIT, MID>(d, from, num_workers, self, at.chunk, tile, kQuads * 4u, kQuads,
                                                        t, lr_local, scale, write_local != 0, lds);
            } else if (tile * kQuads < d.ext.tail_bytes) {
                // (the packed bytes of the ragged end cover its elements: tiles past them have nothing to do)
                const unsigned elems0 = tile * kQuads * 4u;
                fused_tile<true, SZ, WAVES, FORM, GT, SPARSE, HOW, WAIT, MID>(d, from, num_workers, self, at.chunk, tile,
                                                       elems_from(elems0, d.ext.tail_elems),
                                                       d.ext.tail_bytes - tile * kQuads, t, lr_local, scale,
                                                       write_local != 0, lds);
            }
        }
        if (num_tiles - b <= grid) break;
        b += grid;
        group_sync<WAVES>();  // the next tile overwrites the LDS block
    }
}

// Passes that use the workers' 32-bit gradients (Alg. 1: WARMUP passes and the
// correction branch of FormalTraining; eq. 1).  No quantisation, residual and
// packed streams are not touched.
//   SUM    true:  the aggregate is summed here from the N gradients, worker order,
//                 own gradient at position `self` (reads 4N + 4, writes 4 or 8 B/element)
//          false: the aggregate is read from agg_full
//   LOCAL  kLocalOnly: eq. 11 alone, w_global untouched (the local half of a split step)
//          kLocalNone: global rule only              (WARMUP, i < n-1)
//          kLocalCopy: w_local = new global weight   (WARMUP, i == n-1, the copy after the pull)
//          kLocalRule: w_local = W - lr_local * g    (WARMUP, i == n; correction passes; eq. 11)
constexpr int kLocalNone = 0, kLocalCopy = 1, kLocalRule = 2;
constexpr int kLocalOnly = 3;  // eq. 11 alone: w_local = W - lr_local * g, the global weights are left alone

// Launch shape of these passes, chosen by measurement: a workgroup is ONE wave that takes one
// quad per lane (a "piece" of 64 quads = 1 KiB of every stream; 16 pieces to a chunk), and the
// N-way sum loads the workers' gradients one after the other, each add waiting for its load.
// Memory-level parallelism comes from the number of waves (20 to 32 per compute unit), not from
// loads in flight per wave: waves that start together then walk the N streams together, so
// the requests in flight chip-wide fall on one or two streams at a time instead of all N.
// On the VGG-16-shaped list with 16 workers the sum runs at 6.2-6.3 TB/s that way; with 15
// loads in flight per wave it ran at 5.6 TB/s, and with 512-lane workgroups, two quads per lane
// and 8 loads in flight at 5.6-5.7 TB/s.  Two at a time, at the residencies launched (lds_of_kernel_sum), are
// worse with 32-bit gradients (VGG-16-shaped, N = 8 / 16: 0.967 / 1.731 ms, 0.918 / 1.631 one at a time; 25 M
// elements, N = 16: 327 and 309 us) and better with 16-bit ones, whose loads are half as large (VGG-16-shaped,
// N = 16: 0.929 ms, 1.148 one at a time; 25 M elements, N = 16: 183 and 204 us; 4 M, N = 8: 20.7 and 21.4 us).
// On short lists there are too few waves for that: with each worker's pointer and gradient waited for in turn the pass took two
// trips to memory a worker, whatever its length.  There kTogether of them are asked for at once, their pointers in one piece
// (sums_together, with the times).
constexpr unsigned kFullBlock = CDSGD_FULL_BLOCK;            // lanes per workgroup = quads per piece
constexpr unsigned kPiecesPerChunk = kChunkQuads / kFullBlock;
constexpr int kInOrder = 0, kTogether = 8;  // IN_FLIGHT
static_assert(kChunkQuads % kFullBlock == 0 && kFullBlock % 64 == 0, "pieces tile a chunk, whole waves");

// One piece of one chunk: quad qi of the chunk for this lane; rem_elems elements of the chunk exist.
// STORE: how the global weights are stored.  kThrough (keeps_results): written through and staying in the memory-side cache,
// where the next pass reads them; the local ones, which no pass reads, are then written through and do not stay.
template <bool G, bool SUM, int LOCAL, int GT, int STORE, int IN_FLIGHT>
__device__ __forceinline__ void full_piece(const TensorDesc &d, const void *const *__restrict__ pg,
                                           int num_peers, int self, size_t quad0, unsigned qi,
                                           unsigned rem_elems, float lr_local, float scale)
{
    float *__restrict__ wg = d.w_global + 4 * quad0;
    float *__restrict__ wl = d.w_local + 4 * quad0;
    const void *__restrict__ grad = grad_at<GT>(d.grad, quad0);
    if (G && 4u * qi >= rem_elems) return;
    const f4 w = ld4g<G>(wg, qi, rem_elems);
    f4 g = {0.0f, 0.0f, 0.0f, 0.0f}, a = {0.0f, 0.0f, 0.0f, 0.0f};
    if (SUM || LOCAL == kLocalRule || LOCAL == kLocalOnly) g = widen<G, GT>(load_grad<G, GT>(grad, qi, rem_elems), rem_elems);
    if (LOCAL == kLocalOnly) {
        f4 vl;
#pragma unroll
        for (unsigned c = 0; c < 4; ++c) vl[c] = __builtin_fmaf(-lr_local, g[c], w[c]);
        st4g<G, STORE>(wl, qi, rem_elems, vl);
        return;
    }
    if (!SUM) a = ld4g<G>(d.agg_full + 4 * quad0, qi, rem_elems);
    if (SUM) {
        const auto load = [&](const void *peer) { return load_grad<G, GT>(grad_at<GT>(peer, quad0), qi, rem_elems); };
        if constexpr (IN_FLIGHT == kInOrder) {
            // 32-bit gradients one at a time, each add waiting for its load, 16-bit ones (half the bytes a load) in pairs:
            // see the note on the launch shape
            const auto add = [&](int p, int end) {
                if (GT != kGradF32)
                    for (; p + 1 < end; p += 2) {
                        const GradQuad<GT> u = load(pg[p]), v = load(pg[p + 1]);
                        a = a + widen<G, GT>(u, rem_elems);
                        a = a + widen<G, GT>(v, rem_elems);
                    }
                for (; p < end; ++p) a = a + widen<G, GT>(load(pg[p]), rem_elems);
            };
            add(0, self);
            a = a + g;
            add(self, num_peers);
        } else {
            for (int p = 0; p < num_peers; p += IN_FLIGHT) {
                const void *peer[IN_FLIGHT];  // fetched in one piece, then all the loads
                GradQuad<GT> u[IN_FLIGHT];
#pragma unroll
                for (int k = 0; k < IN_FLIGHT; ++k) peer[k] = pg[p + k < num_peers ? p + k : num_peers - 1];
#pragma unroll
                for (int k = 0; k < IN_FLIGHT; ++k) asm volatile("" : "+s"(peer[k]));
#pragma unroll
                for (int k = 0; k < IN_FLIGHT; ++k)
                    if (p + k < num_peers) u[k] = load(peer[k]);
#pragma unroll
                for (int k = 0; k < IN_FLIGHT; ++k)
                    if (p + k < num_peers) {
                        if (p + k == self) a = a + g;
                        a = a + widen<G, GT>(u[k], rem_elems);
                    }
            }
            if (self == num_peers) a = a + g;
        }
    }
    f4 vg, vl;
#pragma unroll
    for (unsigned c = 0; c < 4; ++c) {
        vg[c] = __builtin_fmaf(-scale, a[c], w[c]);
        vl[c] = LOCAL == kLocalRule ? __builtin_fmaf(-lr_local, g[c], w[c]) : vg[c];
    }
    if (LOCAL != kLocalNone) st4g<G, STORE == kThrough ? kThroughStream : STORE>(wl, qi, rem_elems, vl);
    st4g<G, STORE>(wg, qi, rem_elems, vg);
}

// peer_grads: [num_tensors][num_peers] pointers (own row left out), or unused when !SUM.
// The grid walks the pieces of the chunk table: piece x belongs to chunk slot x / kPiecesPerChunk.
template <bool SUM, int LOCAL, int GT, int STORE, int IN_FLIGHT>
__global__ __launch_bounds__(CDSGD_FULL_BLOCK) void k_fused_full(const TensorDesc *__restrict__ tensors,
                                                                 const ChunkRef *__restrict__ chunks,
                                                                 unsigned long long num_pieces,
                                                                 const void *const *__restrict__ peer_grads,
                                                                 int num_peers, int self, float lr_local,
                                                                 float scale)
{
    for (unsigned long long b = blockIdx.x; b < num_pieces; b += gridDim.x) {
        const unsigned long long x = piece_of_workgroup<CDSGD_XCD_FULL != 0>(b, kPiecesPerChunk, num_pieces);
        const ChunkRef cr = chunks[x / kPiecesPerChunk];
        const TensorDesc d = tensors[cr.tensor];
        const size_t quad0 = (size_t)cr.chunk * kChunkQuads;
        const unsigned qi = (unsigned)(x % kPiecesPerChunk) * kFullBlock + threadIdx.x;
        const void *const *pg = SUM ? peer_grads + (size_t)cr.tensor * (size_t)num_peers : nullptr;
        if (cr.chunk < d.ext.full_chunks)
            full_piece<false, SUM, LOCAL, GT, STORE, IN_FLIGHT>(d, pg, num_peers, self, quad0, qi, kChunkElems, lr_local, scale);
        else
            full_piece<true, SUM, LOCAL, GT, STORE, IN_FLIGHT>(d, pg, num_peers, self, quad0, qi, d.ext.tail_elems, lr_local, scale);
    }
}

}  // namespace
