// Decode-and-sum of the workers' packed streams for one tile (a4: Sec. 3.2.1; the sum of eq. 10).
#pragma once

namespace {

// A tile is 1024 elements of a tensor, the work of a group of four waves: 4 KiB of every fp32 stream, one quad per
// lane (quad 64 v + l for lane l of wave v), and 256 bytes of every packed stream, two whole 128-byte lines, 64
// words.  The group decodes words, sixteen consecutive elements each, not the bytes of a lane's own quad.
constexpr unsigned kTileQuads = 256, kTileWords = 64, kTileBytes = kTileQuads;
constexpr unsigned kTilesPerChunk = kChunkQuads / kTileQuads;
static_assert(kChunkQuads % kTileQuads == 0, "tiles tile a chunk");

// How a kernel is compiled for the number of workers.  The waves share the workers out: wave v takes
// kWordsPerWave<SZ> of every row, lane l its word l of each, and all of a group's loads are in flight at once.
constexpr int kUpTo4 = 4, kUpTo8 = 8, kUpTo16 = 16, kUpTo32 = 32, kAnyWorkers = 0;
template <int SZ>
constexpr int kMaxRows = SZ == kAnyWorkers ? CDSGD_MAX_WORKERS : SZ;
template <int SZ>
constexpr int kWordsPerWave = kMaxRows<SZ> / 4;

typedef unsigned u4 __attribute__((ext_vector_type(4)));

// values of the codes of a register, as 2-bit two's-complement fields (01 -> +1, 10 -> -1, else 0): the low bit is low ^ high,
// the high bit high & ~low.
__device__ __forceinline__ unsigned signed_fields(unsigned w)
{
    constexpr unsigned kLow = 0x55555555u;
    const unsigned low = __builtin_amdgcn_bitop3_b32(w, w >> 1, kLow, 0x28);    // (w ^ w >> 1) & kLow
    return __builtin_amdgcn_bitop3_b32(low, w, (w << 1) | kLow, 0xF4);          // low | w & ~(w << 1 | kLow)
}

// A row of stream pointers: one entry per worker, in worker order, null where there is nothing to load (the own
// entry, and the entries past the last worker up to a whole batch).
inline constexpr unsigned row_entries(int num_workers)
{
    return num_workers <= kUpTo8 ? 8u : ((unsigned)num_workers + 15u) / 16u * 16u;
}

// Decode forms.  kCount: thresholds that are powers of two, where every partial sum is exact and the sum is
// count x t bit for bit.  kChain: one rounded add per worker and element, in worker order.  kChainTiny: the same
// for thresholds below 2^-125, whose half may not be exact (the passes over a list have it for any number of workers only).
constexpr int kCount = 0, kChain = 1, kChainTiny = 2;

// One word of a buffer of `bytes` bytes at byte offset `off`; 0 past the end (the buffer's own range check), which
// is what the lanes behind a ragged end and the absent workers (bytes == 0: nothing is read) want.
// POLICY: 0, or kStream where the streams are more than the caches hold (load_packed).
template <int POLICY>
__device__ __forceinline__ unsigned ld_word(const uint8_t *base, unsigned bytes, unsigned off)
{
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, (int)bytes, kBufferFlags);
    return __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off, 0, POLICY);
}

// Where the streams of a tile are.
struct TileStreams {
    int num_workers;
    unsigned stream_bytes;      // packed form: bytes of a stream, and where the tile starts in it
    unsigned tile_at;
    size_t segment_at;          // sparse form: the chunk's segment, and the tile's number in the chunk
    unsigned tile;
};

// The worker whose word a wave holds in slot i: four neighbours out of every sixteen (two out of eight, one out of
// four), so that the slots of a wave fill up evenly with the number of workers.
template <int SZ>
__device__ __forceinline__ constexpr int worker_of(int wave, int i)
{
    return SZ == kUpTo4 ? wave : (SZ == kUpTo8 ? 2 * wave + i : 16 * (i / 4) + 4 * wave + i % 4);
}

// The streams of the workers that a wave takes (a group of one wave: that the lane takes); null: nothing to load.
// They are fetched in one piece and before anything waits: a load that stands inside the test for its worker is
// fetched, waited for and used before the next, which cost the kernels for more than 16 workers up to 16 trips to
// the scalar cache in a row, and behind the descriptor of the tensor it costs every group one trip.
template <int SZ, int WAVES, bool SPARSE>
struct StreamPointers {
    const uint8_t *p[kWordsPerWave<SZ>];
    const uint8_t *bitmap;  // sparse form: the stream of the worker whose bitmap words the lane fetches

    // `row` has row_entries(num_workers) entries, and kMaxRows<SZ> can be read.  SELECT: the lanes pick the bitmap's
    // stream from the wave's pointers instead of reading it from the row, which is a trip to memory of its own where
    // the row is in the kernel's arguments (decode-and-sum of 2^27 elements, sparse, N = 4 and 8, one code in 256:
    // 1.09 and 1.07 against 0.97 and 1.00 of the time of a kernel that stages the bitmaps through LDS).
    template <bool SELECT>
    __device__ __forceinline__ void load(const uint8_t *const *__restrict__ row, int num_workers, int wave, unsigned lane)
    {
        bitmap = nullptr;
        if constexpr (WAVES == 1) {
            static_assert(SZ == kUpTo8 && !SPARSE, "one wave: up to eight packed streams");
#pragma unroll
            for (int i = 0; i < kWordsPerWave<SZ>; ++i) p[i] = row[2u * (lane >> 4) + (unsigned)i];
        } else {
#pragma unroll
            for (int i = 0; i < kWordsPerWave<SZ>; ++i) p[i] = row[worker_of<SZ>(wave, i)];
            if constexpr (SPARSE) {
                const int slot = (int)(lane >> 2);
                if constexpr (SELECT && SZ != kAnyWorkers) {
#pragma unroll
                    for (int i = 0; i < kWordsPerWave<SZ>; ++i)
                        if (slot == i) bitmap = p[i];
                } else if (slot < kWordsPerWave<SZ>) {
                    const int j = worker_of<SZ>(wave, slot);
                    if (SZ != kAnyWorkers || j < num_workers) bitmap = row[j];
                }
            }
        }
    }

    // Keeps the compiler from moving the loads to where their pointers are used.  Above 32 workers a wave of the fused
    // kernels then needs all 106 scalar registers, which admit six groups to a compute unit (kSix); with sparse peers, which
    // have more addresses, 10 (count form) and 13 to 15 (chain) of them are kept in lanes of a vector register, and in the
    // form for tiny thresholds 1.
    // Short lists, where the early pointers count, gain all the same (figures at the head of kernels_fused.hpp); long
    // ones run no better with more groups.  The single-tensor decode has no descriptor and spills none.
    __device__ __forceinline__ void pin()
    {
        if constexpr (WAVES != 1) {
#pragma unroll
            for (int i = 0; i < kWordsPerWave<SZ>; ++i) asm volatile("" : "+s"(p[i]));
        }
    }
};

// This lane's words of the workers that its wave takes; 0 where there is nothing to load.
// NT: non-temporal.  A bare read of 32 streams of 4 MB beside one written: 38.7 us at the default policy, 33.6 so.
template <int SZ, bool NT>
__device__ __forceinline__ void load_packed(unsigned (&w)[kWordsPerWave<SZ>], const uint8_t *const (&p)[kWordsPerWave<SZ>],
                                            const TileStreams &s, int wave, unsigned lane)
{
#pragma unroll
    for (int i = 0; i < kWordsPerWave<SZ>; ++i) {
        const bool there = p[i] && (SZ != kAnyWorkers || worker_of<SZ>(wave, i) < s.num_workers);
        w[i] = ld_word<NT ? kStream : 0>(p[i], there ? s.stream_bytes : 0u, s.tile_at + 4u * lane);
    }
}

// The same from streams in the sparse form (segment of 8 bitmap words and the non-zero words, see kernels_sparse.hpp).
// Lane 4 i + m fetches bitmap words 2 m and 2 m + 1 of the worker in slot i; a tile's 64 words are one such pair, so
// its bitmap, and the number of words in front of it, are wave-uniform, and a lane's word lies at the rank of its bit.
// The bitmap words are the chunk's, the same for each of its tiles.
__device__ __forceinline__ u2 load_bitmap(const uint8_t *stream, const TileStreams &s, unsigned lane)
{
    u2 bm = {0u, 0u};
    typedef unsigned u2a __attribute__((ext_vector_type(2), aligned(4)));
    if (stream) bm = *(const CDSGD_GLOBAL u2a *)(stream + s.segment_at + 8u * (lane & 3u));
    return bm;
}

template <int SZ>
__device__ __forceinline__ void load_sparse(unsigned (&w)[kWordsPerWave<SZ>], const StreamPointers<SZ, 4, true> &from,
                                            u2 bm, const TileStreams &s, int wave, unsigned lane)
{
    const unsigned m = lane & 3u;
    // words in front of the tile's own: summed over the worker's four lanes
    int before = m < s.tile ? __builtin_popcount(bm.x) + __builtin_popcount(bm.y) : 0;
    before += __builtin_amdgcn_mov_dpp(before, 0xB1, 0xF, 0xF, true);  // quad_perm [1, 0, 3, 2]
    before += __builtin_amdgcn_mov_dpp(before, 0x4E, 0xF, 0xF, true);  // quad_perm [2, 3, 0, 1]
#pragma unroll
    for (int i = 0; i < kWordsPerWave<SZ>; ++i) {
        w[i] = 0u;
        if (SZ != kAnyWorkers || 16 * (i / 4) < s.num_workers) {
            const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)bm.x, 4 * i + (int)s.tile);
            const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)bm.y, 4 * i + (int)s.tile);
            const unsigned at = 8u + (unsigned)__builtin_amdgcn_readlane(before, 4 * i);
            const uint8_t *p = from.p[i];
            const unsigned rank = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
            const bool sent = __builtin_amdgcn_inverse_ballot_w64(((unsigned long long)hi << 32) | lo);
            // a lane whose word is zero asks past the end of the segment and gets 0 without a read
            const bool there = p && (SZ != kAnyWorkers || worker_of<SZ>(wave, i) < s.num_workers);
            w[i] = ld_word<0>(p + s.segment_at, there ? 4u * kSegStride : 0u, sent ? 4u * (at + rank) : 4u * kSegStride);
        }
    }
}

// Groups of one wave: a quarter of a tile, 16 words of every stream; lanes 16 v .. 16 v + 15 take what wave v takes
// in a group of four (packed form, up to eight workers).
__device__ __forceinline__ void load_packed_quarter(unsigned (&w)[kWordsPerWave<kUpTo8>],
                                                    const uint8_t *const (&p)[kWordsPerWave<kUpTo8>],
                                                    const TileStreams &s, unsigned lane)
{
    const unsigned off = s.tile_at + 4u * (lane & 15u);
#pragma unroll
    for (int i = 0; i < kWordsPerWave<kUpTo8>; ++i) {
        w[i] = 0u;
        if (p[i] && off < s.stream_bytes) w[i] = *global_ptr(reinterpret_cast<const unsigned *>(p[i] + off));
    }
}

template <int SZ, int WAVES, bool SPARSE, bool NT>
__device__ __forceinline__ void load_words(unsigned (&w)[kWordsPerWave<SZ>], const StreamPointers<SZ, WAVES, SPARSE> &from,
                                           const TileStreams &s, int wave, unsigned lane)
{
    if constexpr (WAVES == 1) load_packed_quarter(w, from.p, s, lane);
    else if constexpr (SPARSE) load_sparse<SZ>(w, from, load_bitmap(from.bitmap, s, lane), s, wave, lane);
    else load_packed<SZ, NT>(w, from.p, s, wave, lane);
}

// ---- count form -------------------------------------------------------------
// Bit-sliced counting.  The value of a code is (low bit) - (high bit), also for the field that is never written
// (11 reads as nothing), so it is enough to count the set bits of the words position by position: a carry-save
// adder is two vector operations (three-input logic) on 32 positions.  Each wave counts its own workers' words, the
// four waves' counts meet in LDS as bytes.  One operation per worker and element, and a byte read from LDS per worker
// and quad, become a tenth of that; with 64 workers that was what bounded the pass (25 M elements: 0.191 ms before,
// 0.169 now, 6.0 TB/s).
__device__ __forceinline__ void csa(unsigned &carry, unsigned &sum, unsigned a, unsigned b, unsigned c)
{
    const unsigned s = __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);  // a ^ b ^ c
    carry = __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);             // at least two of the three
    sum = s;
}

template <int PLANES>
struct BitCounts {
    unsigned p[PLANES];  // p[i]: bit i of the count of every position

    // Count W words (W = 1, 2, 4, 8 or 16; at most 2^PLANES - 1 at a time can be held).
    template <int W>
    __device__ __forceinline__ void count(const unsigned (&w)[W])
    {
        if constexpr (W == 1) {
            p[0] = w[0];
        } else if constexpr (W == 2) {
            p[0] = w[0] ^ w[1];
            p[1] = w[0] & w[1];
        } else {
            static_assert(W % 4 == 0, "words in groups of four");
#pragma unroll
            for (int i = 0; i < PLANES; ++i) p[i] = 0u;
#pragma unroll
            for (int i = 0; i < W; i += 4) {
                unsigned t0, t1, e;
                csa(t0, p[0], p[0], w[i], w[i + 1]);
                csa(t1, p[0], p[0], w[i + 2], w[i + 3]);
                csa(e, p[1], p[1], t0, t1);
#pragma unroll
                for (int k = 2; k < PLANES; ++k) {
                    const unsigned both = p[k] & e;
                    p[k] ^= e;
                    e = both;
                }
            }
        }
    }

    // Byte j of out[c] = (2^PLANES - 1) + sum of the values of element 4 j + c of the lane's word.
    __device__ __forceinline__ void to_bytes(unsigned (&out)[4]) const
    {
        static_assert(PLANES <= 5, "four groups' fields, 2^PLANES - 1 plus a count each, add up in a byte");
#pragma unroll
        for (int i0 = 0; i0 < PLANES; i0 += 3) {
            unsigned even = 0u, odd = 0u;  // nibbles: elements 0, 2, 4, ... and 1, 3, 5, ...; three planes: at most 14
#pragma unroll
            for (int i = i0; i < i0 + 3 && i < PLANES; ++i) {
                // 1 + (low bit) - (high bit) of every position pair, in the pair's two bits
                const unsigned h = p[i] >> 1;
                const unsigned same = __builtin_amdgcn_bitop3_b32(p[i], h, 0x55555555u, 0x82);  // ~(p ^ h) & mask
                const unsigned plus = __builtin_amdgcn_bitop3_b32(p[i], h, 0x55555555u, 0x20);  // p & ~h & mask
                const unsigned z = (plus << 1) | same;
                even += (z & 0x33333333u) << (i - i0);
                odd += ((z >> 2) & 0x33333333u) << (i - i0);
            }
            const unsigned b0 = even & 0x0F0F0F0Fu, b2 = (even >> 4) & 0x0F0F0F0Fu;
            const unsigned b1 = odd & 0x0F0F0F0Fu, b3 = (odd >> 4) & 0x0F0F0F0Fu;
            out[0] = i0 == 0 ? b0 : out[0] + (b0 << i0);
            out[1] = i0 == 0 ? b1 : out[1] + (b1 << i0);
            out[2] = i0 == 0 ? b2 : out[2] + (b2 << i0);
            out[3] = i0 == 0 ? b3 : out[3] + (b3 << i0);
        }
    }
};

// planes a wave needs: counts up to 1, 2, 4, 8 and 16
template <int SZ>
constexpr int kPlanes = SZ == kUpTo4 ? 1 : (SZ == kUpTo8 ? 2 : (SZ == kUpTo16 ? 3 : (SZ == kUpTo32 ? 4 : 5)));

// ---- chain form -------------------------------------------------------------
// One rounded add of +t, -t or 0 per worker and element: a fused multiply-add whose multiplier is a 16-bit float
// read from half a register.  The top two bits of a 16-bit float are its sign and the top bit of its exponent:
// 01 is +2, 11 is -2 and 00 is 0, which is the two's-complement form of a code's value.  So a word's codes become
// multipliers with one shift and one mask for two elements, and the products are exact with t / 2.
// The half of a threshold below 2^-125 is not exact if its last bit is odd.  Such sums (kChainTiny) are formed 2^64 times
// as large and scaled back at the end, which changes no bit: every term and partial sum is a multiple of 2^-149, so
// those below 2^-125 are exact in either place and those above are normal numbers in both.
// A bit more than 2 vector operations per worker and element, against 4.25 with a bit-field extract, a convert and a
// multiply-add per element of every byte (25 M elements, N = 64, bf16 gradients: 0.226 ms before, 0.164 now).
typedef _Float16 h2 __attribute__((ext_vector_type(2)));

// Two of a word's eight pairs: elements i and i + 8, i + 1 and i + 9, from the word's signed fields; shift = 14 - 2 i.
__device__ __forceinline__ void chain_pairs(float (&acc)[4], unsigned fields, unsigned shift, float t)
{
    const float factor = 0.5f * t;
    const h2 a = __builtin_bit_cast(h2, (fields << shift) & 0xC000C000u);
    const h2 b = __builtin_bit_cast(h2, (fields << (shift - 2u)) & 0xC000C000u);
    acc[0] = __builtin_fmaf((float)a.x, factor, acc[0]);
    acc[1] = __builtin_fmaf((float)b.x, factor, acc[1]);
    acc[2] = __builtin_fmaf((float)a.y, factor, acc[2]);
    acc[3] = __builtin_fmaf((float)b.y, factor, acc[3]);
}

// A quad's four codes, from the byte of signed fields.
__device__ __forceinline__ void chain_byte(f4 &acc, unsigned byte, float t)
{
    const float factor = 0.5f * t;
    const unsigned y = (byte << 12) | (byte << 24);
    const h2 a = __builtin_bit_cast(h2, (y << 2) & 0xC000C000u);  // elements 0 and 2
    const h2 b = __builtin_bit_cast(h2, y & 0xC000C000u);         // elements 1 and 3
    acc[0] = __builtin_fmaf((float)a.x, factor, acc[0]);
    acc[1] = __builtin_fmaf((float)b.x, factor, acc[1]);
    acc[2] = __builtin_fmaf((float)a.y, factor, acc[2]);
    acc[3] = __builtin_fmaf((float)b.y, factor, acc[3]);
}

// ---- a tile's sums ------------------------------------------------------------
// LDS of a group: the four waves' partial counts, or the workers' words as signed fields and the sums on their way
// from words to quads.
// Chain form: up to 16 workers every lane adds up the bytes of its own quad, above that the lanes add up words and
// exchange the sums (decode-and-sum of 2^27 elements, N = 32: 0.270 ms by words, 0.298 by bytes).
template <int SZ>
constexpr bool kByBytes = SZ != kAnyWorkers && SZ <= kUpTo16;
template <int SZ, bool SPARSE>
constexpr bool kSlotTests = SPARSE || SZ == kUpTo4 || SZ == kUpTo8;  // tile_put
template <int SZ>
constexpr unsigned kSpareRow = (unsigned)kMaxRows<SZ>;  // written and not read; where there are sums they follow later
// SPARE: there is an own row that is not tested for (tile_put).
template <int SZ, bool SPARE>
constexpr unsigned kRowsLds = (unsigned)kMaxRows<SZ> * kTileBytes + (!kByBytes<SZ> ? 16u * kTileQuads : (SPARE ? kTileBytes : 0u));
template <int SZ, int FORM, int WAVES, bool SPARSE, bool OWN>
constexpr unsigned kTileLds = (FORM == kCount ? 4u * 4u * kTileQuads : kRowsLds<SZ, OWN && !kSlotTests<SZ, SPARSE>>) * WAVES / 4;

template <int WAVES>
__device__ __forceinline__ void group_sync()
{
    if (WAVES == 1) {
        // one wave's LDS operations run in order, only the compiler has to keep them so
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// A lane's place in its group.  A group of four waves: wave v holds words of its workers, word l in lane l; a group of
// one: lanes 16 v ..
template <int WAVES>
struct TilePlace {
    unsigned tid, lane;
    int wave;
    __device__ __forceinline__ TilePlace()
    {
        tid = threadIdx.x;
        lane = tid & (16u * WAVES - 1u);
        wave = WAVES == 4 ? __builtin_amdgcn_readfirstlane((int)(tid >> 6)) : (int)(tid >> 4);
    }
};

// The sums of this lane's quad of a tile over all workers.  `w` holds the wave's words (load_words); the own codes
// come as this lane's packed byte and as the values it stands for, own_at is their place in the order (-1: none).
// In two halves, with a barrier between them: the first leaves in LDS what the waves know of their workers, the second
// reads it.  Everything a group has written to LDS before has been read when it starts over (a barrier of the caller's).
template <int SZ, int FORM, int WAVES, bool TESTS>
__device__ __forceinline__ void tile_put(const unsigned (&w)[kWordsPerWave<SZ>], unsigned own_code, int own_at,
                                         int num_workers, uint8_t *lds, TilePlace<WAVES> at)
{
    constexpr unsigned kWords = 16u * WAVES, kBytes = 64u * WAVES;
    const unsigned tid = at.tid, lane = at.lane;
    const int wave = at.wave;
    if (FORM == kCount) {
        constexpr int P = kPlanes<SZ>;
        BitCounts<P> counts;
        counts.count(w);
        unsigned a[4];
        counts.to_bytes(a);
        // a[c] byte j -> dword j byte c: one dword per quad of this lane's word
        const unsigned x0 = __builtin_amdgcn_perm(a[1], a[0], 0x05010400u), x1 = __builtin_amdgcn_perm(a[1], a[0], 0x07030602u);
        const unsigned y0 = __builtin_amdgcn_perm(a[3], a[2], 0x05010400u), y1 = __builtin_amdgcn_perm(a[3], a[2], 0x07030602u);
        u4 q;
        q[0] = __builtin_amdgcn_perm(y0, x0, 0x05040100u);
        q[1] = __builtin_amdgcn_perm(y0, x0, 0x07060302u);
        q[2] = __builtin_amdgcn_perm(y1, x1, 0x05040100u);
        q[3] = __builtin_amdgcn_perm(y1, x1, 0x07060302u);
        reinterpret_cast<u4 *>(lds)[tid] = q;  // [wave][word][quad]
    } else {
        // Rows of signed fields, worker by worker; those past the last worker are zero.  Packed streams of more than eight
        // workers: every slot is written without a test.  Behind a test of its own (a slot past the last worker, the own one) the compiler puts the load of
        // the slot's word as well, as it sees fit, and a wave of the kernels for any number of workers then waits for memory twice.
        // With tests / so, us: 16.7 M elements decoded and updated, t = 0.3, N = 33 / 48 / 64 80.3 / 87.5 / 103.0, 66.5 / 77.5 / 90.1;  4 M
        // 21.9 / 24.4 / 29.0, 19.0 / 22.3 / 25.7;  compressed pass 0.5 M N = 32 / 64 4.3 / 6.5, 4.2 / 6.1;  1 M 7.1 / 9.9, 6.7 / 9.5;
        // 4 M 21.4 / 28.2, 21.4 / 27.7.  (With tests and the fields made without bitop3 the decode waited once: 67.1 / 78.2 /
        // 91.4 and 19.5 / 22.8 / 26.6.)  The own row is made of the lanes' own codes; what the wave holds for it goes to
        // the spare row.  (Sparse streams, whose words have to wait for their bitmaps: N = 64 2-6 % faster without tests, 33 to 48
        // 1-5 % slower; packed streams of 5 to 8 workers, 60 M elements 1 % slower.  MID of the compressed pass: there.)
        unsigned *rows = reinterpret_cast<unsigned *>(lds);
#pragma unroll
        for (int i = 0; i < kWordsPerWave<SZ>; ++i) {
            const int j = worker_of<SZ>(wave, i);
            if constexpr (TESTS) {
                if (j != own_at && (SZ != kAnyWorkers || 16 * (i / 4) < num_workers)) rows[kWords * (unsigned)j + lane] = signed_fields(w[i]);
            } else {
                rows[kWords * (j != own_at ? (unsigned)j : kSpareRow<SZ>) + lane] = signed_fields(w[i]);
            }
        }
        if (own_at >= 0) lds[kBytes * (unsigned)own_at + tid] = (uint8_t)signed_fields(own_code);
    }
}

// READS, chain form up to 16 workers: kOneTest: all rows behind one test;  kAllFirst: all read in front of the tests;  0: as the compiler has them.
constexpr int kOneTest = 1, kAllFirst = 2;
template <int SZ, int FORM, int WAVES, bool SPREAD, int READS>
__device__ __forceinline__ f4 tile_get(f4 own_value, int num_workers, float t, uint8_t *lds, TilePlace<WAVES> at)
{
    constexpr unsigned kQuads = 64u * WAVES, kBytes = kQuads;
    const unsigned tid = at.tid, lane = at.lane;
    const int wave = at.wave;
    f4 agg;
    if (FORM == kCount) {
        constexpr int P = kPlanes<SZ>;
        unsigned v = 0u;
#pragma unroll
        for (unsigned k = 0; k < 4; ++k) v += reinterpret_cast<const unsigned *>(lds)[kQuads * k + tid];
        const float bias_t = -(float)(4 * ((1 << P) - 1)) * t;
#pragma unroll
        for (unsigned c = 0; c < 4; ++c) agg[c] = __builtin_fmaf((float)((v >> (8u * c)) & 0xFFu), t, bias_t);
        agg = agg + own_value;
    } else {
        const unsigned *rows = reinterpret_cast<const unsigned *>(lds);
        const bool tiny = FORM == kChainTiny && t < 0x1p-125f;  // (a list's own thresholds may be of either kind)
        if (tiny) t *= 0x1p64f;
        if constexpr (kByBytes<SZ>) {
            // every lane adds up its own quad, a byte of every row: one operation more per worker than by words, no exchange
            agg = f4{0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (READS == kOneTest) {
                // One test and then all rows, their bytes read at once.  With a test for every four rows the compiler puts the reads
                // behind it as well, or in front of all of them, as it sees fit: a trip to LDS for every four rows.  Decode-and-sum,
                // t = 0.1, time over that, 1 / 1.6 / 2.2 / 3 / 6 / 16 M elements (in the other kernels the reads are in front, of up to 8 workers half of them):
                //   packed  N = 9 and 12 .89 .95 .95 .94 .96 .99;  13 .92 .95 .97 .97 .99 1.00;  16 .93 .96 .98 .99 .99 1.00;  5 and 8, 2 to 16 M .96-.99
                //   sparse  3 to 16 M  N = 2 and 4 .98-.99;  8 .97-1.00  (9 to 12, 1 to 16 M .92-1.00, but 13 and 16 from 6 M on 1.01-1.03)
                const auto add = [&](auto rows) {
                    constexpr int ROWS = decltype(rows)::value;
                    unsigned code[ROWS];
#pragma unroll
                    for (int j = 0; j < ROWS; ++j) code[j] = lds[kBytes * (unsigned)j + tid];
#pragma unroll
                    for (int j = 0; j < ROWS; ++j) chain_byte(agg, code[j], t);
                };
                if (SZ == kUpTo16 && num_workers <= 12) add(std::integral_constant<int, 12 < SZ ? 12 : SZ>{});
                else add(std::integral_constant<int, SZ>{});
            } else {
                unsigned code[SZ];
#pragma unroll
                for (int j = 0; j < SZ; ++j) code[j] = lds[kBytes * (unsigned)j + tid];
                if constexpr (READS == kAllFirst) {
#pragma unroll
                    for (int j = 0; j < SZ; ++j) asm volatile("" : "+v"(code[j]));
                }
#pragma unroll
                for (int j0 = 0; j0 < SZ; j0 += 4)
                    if (j0 < num_workers) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) chain_byte(agg, code[j0 + k], t);
                    }
            }
        } else {
            float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            const unsigned shift = 14u - 4u * (unsigned)wave;
            for (int j0 = 0; j0 < num_workers; j0 += 4) {
#pragma unroll
                for (int k = 0; k < 4; ++k) chain_pairs(acc, rows[kTileWords * (j0 + k) + lane], shift, t);
            }
            // Elements 2 v, 2 v + 1 and 2 v + 8, 2 v + 9 of word l -> quads.  SPREAD: word l's four quads lie in an order that goes
            // by l / 4; in plain order the lanes of a wave write to an eighth of the banks.  Time spread over plain: decode and
            // update, sparse streams, t = 0.3 1.5 M elements N = 17 / 24 / 32 / 64 .98 / .97 / .97 / .99, 4 M .99, 16.7 and 40 M .99-1.00;
            // compressed pass N = 32 0.5 M .96, bf16 .98, 4 M .99, N = 64 0.5 M .96, bf16 .95, 1 M .98, 12 and 25 M 1.00.  Packed streams
            // of a single tensor keep the plain order: 1.5 M .98-1.00, but 8 to 40 M 1.01-1.03 (with rows 20 floats apart the
            // same): their groups are through sooner, and the order in which memory is asked is the worse one.
            typedef float f2 __attribute__((ext_vector_type(2)));
            float *sums = reinterpret_cast<float *>(lds + (unsigned)kMaxRows<SZ> * kTileBytes);
            const unsigned quad = 4u * lane + (((unsigned)wave >> 1) ^ (SPREAD ? lane >> 2 & 3u : 0u)), half = 2u * ((unsigned)wave & 1u);
            *reinterpret_cast<f2 *>(sums + 4u * quad + half) = f2{acc[0], acc[1]};
            *reinterpret_cast<f2 *>(sums + 4u * (quad ^ 2u) + half) = f2{acc[2], acc[3]};
            group_sync<WAVES>();
            agg = reinterpret_cast<const f4 *>(sums)[tid ^ (SPREAD ? tid >> 4 & 3u : 0u)];
        }
        if (tiny) agg = agg * 0x1p-64f;
    }
    return agg;
}

template <int SZ, int FORM, int WAVES, bool TESTS, bool SPREAD, int READS>
__device__ __forceinline__ f4 tile_sums(const unsigned (&w)[kWordsPerWave<SZ>], unsigned own_code, f4 own_value,
                                        int own_at, int num_workers, float t, uint8_t *lds)
{
    const TilePlace<WAVES> at;
    tile_put<SZ, FORM, WAVES, TESTS>(w, own_code, own_at, num_workers, lds, at);
    group_sync<WAVES>();
    return tile_get<SZ, FORM, WAVES, SPREAD, READS>(own_value, num_workers, t, lds, at);
}

// ---------------------------------------------------------------------------
// a4 for one tensor, packed or sparse streams: TILES tiles of a chunk per group of four waves
// ---------------------------------------------------------------------------
// Bound by HBM (4 + N / 4 bytes per element), as long as a group has enough to load and store: with few workers one
// tile a group is too little (each group lives for one or two round trips, the sparse form's bitmaps in front of its
// words), so the loads of TILES tiles are in flight together and one barrier serves them all; a chunk's bitmaps are
// fetched once.  Time of the call, 2^27 elements, several sets of buffers in turn, us: a kernel that takes a chunk per
// group and stages bytes through LDS / one tile a group / now (the TILES of launch_decode_sum):
//   packed   N = 2 108 / 133 / 96;  4 106 / 138 / 110;  8 128 / 139 / 126;  17, t = 0.3 212 / 227 / 201
//   sparse, one code in 4     N = 4 112 / 238 / 114;  8 139 / 237 / 142;  16 194 / 242 / 201;  17 216 / 280 / 209
//   sparse, one code in 256   N = 4 103 / 183 / 100;  8 146 / 248 / 146;  16 194 / 267 / 184;  17 221 / 292 / 209
// With many workers it is the word-wise decode that pays (2^24 elements, N = 32 and 64, t = 0.3: 55 and 100 us with
// the chunk-wise kernel, 40 and 65 now).
// xcd: which order the tiles are dealt in.  The chunk-wise order pays where the tiles of a chunk share its segment
// (sparse streams), and on long tensors (2^27 elements, N = 16: 421 against 428 us); on shorter ones the plain order
// is 1 % faster (2^24: 71.5 against 72.5; both with the global update behind it).
// drain: the aggregate is stored non-temporally (drains_results).  Otherwise it is written through and stays in the
// memory-side cache, where the global update that follows finds it (decode-and-sum and update, non-temporal store / now,
// us: N = 16, 50 M 162 / 150; N = 32, 16 M 70 / 66; N = 4, 4 M 13.0 / 12.5; at the default policy the flush of the L2s at
// the end of the kernel costs what the update gains).
// The workers' stream pointers of a single-tensor call; they travel in the kernel arguments.
struct StreamTable {
    const uint8_t *p[CDSGD_MAX_WORKERS];  // null past the last worker
};

template <int SZ, int FORM, bool SPARSE, int TILES, bool NT>
__global__ __launch_bounds__(kTileQuads) void k_decode_sum(float *__restrict__ agg_out, Extent ext, int num_workers,
                                                           unsigned num_groups, int xcd, int drain, float t, StreamTable tab)
{
    static_assert(kTilesPerChunk % TILES == 0, "the tiles of a group lie in one chunk");
    constexpr unsigned kPerChunk = kTilesPerChunk / TILES, kLds = kTileLds<SZ, FORM, 4, SPARSE, false>;
    __shared__ __attribute__((aligned(16))) uint8_t lds[kLds * TILES];
    const unsigned tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane((int)(tid >> 6));
    const unsigned x = xcd ? piece_of_workgroup<true>(blockIdx.x, kPerChunk, num_groups) : blockIdx.x;
    const unsigned chunk = x / kPerChunk;
    StreamPointers<SZ, 4, SPARSE> from;
    from.template load<true>(tab.p, num_workers, wave, tid & 63u);
    from.pin();
    TileStreams s;
    s.num_workers = num_workers;
    s.stream_bytes = ext.full_chunks * kChunkQuads + ext.tail_bytes;
    s.segment_at = (size_t)chunk * (4u * kSegStride);
    u2 bitmap = {0u, 0u};
    if constexpr (SPARSE) bitmap = load_bitmap(from.bitmap, s, tid & 63u);
    const TilePlace<4> at;
    unsigned words[TILES][kWordsPerWave<SZ>];
#pragma unroll
    for (unsigned k = 0; k < TILES; ++k) {
        s.tile_at = (x * TILES + k) * kTileBytes;
        s.tile = x % kPerChunk * TILES + k;
        if constexpr (SPARSE) load_sparse<SZ>(words[k], from, bitmap, s, wave, tid & 63u);
        else load_packed<SZ, NT>(words[k], from.p, s, wave, tid & 63u);
    }
#pragma unroll
    for (unsigned k = 0; k < TILES; ++k) tile_put<SZ, FORM, 4, kSlotTests<SZ, SPARSE>>(words[k], 0u, -1, num_workers, lds + kLds * k, at);
    group_sync<4>();
    float *out = agg_out + (size_t)x * (4u * kTileQuads * TILES);
#pragma unroll
    for (unsigned k = 0; k < TILES; ++k) {
        const f4 agg = tile_get<SZ, FORM, 4, SPARSE, !SPARSE || SZ == kUpTo4 || SZ == kUpTo8 ? kOneTest : 0>(f4{0.0f, 0.0f, 0.0f, 0.0f}, num_workers, t, lds + kLds * k, at);
        const unsigned qi = kTileQuads * k + tid;
        if (chunk < ext.full_chunks) {
            if (drain) st4p<kStream>(out, qi, agg);
            else st4p<kThrough>(out, qi, agg);
        } else {
            const unsigned e0 = x % kPerChunk * (4u * kTileQuads * TILES);
            st4g<true, kThrough>(out, qi, elems_from(e0, ext.tail_elems), agg);
        }
    }
}

}  // namespace
