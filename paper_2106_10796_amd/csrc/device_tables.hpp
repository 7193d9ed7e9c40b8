// Device-side tables of a layer list: extents, tensor descriptors, chunk table.
#pragma once

namespace {

// ---------------------------------------------------------------------------
// device-side tables of a plan
// ---------------------------------------------------------------------------
// How a tensor of n elements splits into chunks: `full_chunks` chunks hold
// kChunkElems elements each; if anything is left, one more chunk holds the
// ragged end: tail_elems elements (< kChunkElems) and tail_bytes bytes of the
// packed stream (the bytes of the last word past the last element included).
// Everything is 32-bit and uniform, so the interior/tail decision is a scalar
// compare on the chunk number.
struct Extent {
    unsigned full_chunks;
    unsigned tail_elems;
    unsigned tail_bytes;
    unsigned pad_;
};

struct TensorDesc {
    float *w_global;
    float *w_local;
    float *residual;
    const void *grad;  // fp32, bf16 or fp16 (the plan's gradient type)
    uint8_t *packed_self;
    const float *agg_full;
    Extent ext;
    float threshold;  // > 0: this tensor's own threshold (cdsgd_plan_set_thresholds); 0: the call's
    unsigned pad_;
};

struct ChunkRef {
    unsigned tensor;  // index into the TensorDesc table
    unsigned chunk;   // chunk number inside that tensor
};

// The same for a list in arenas: every buffer of a tensor lies as far from tensor 0's as every other (in elements), and
// a chunk is found from tensor 0's buffers without a look at its tensor's descriptor.
struct ArenaChunk {
    unsigned off16;  // the chunk's first element, counted from tensor 0's first in units of 16
    unsigned elems;  // elements of the chunk
};
static_assert(sizeof(ArenaChunk) == sizeof(ChunkRef), "either kind of entry fits a chunk table");

// Every kernel over a layer list walks the pieces of the chunk table from its workgroup number
// in steps of the grid size.  Normally the grid has one workgroup per piece and the loop runs
// once; a plan with a workgroup limit (cdsgd_plan_set_max_workgroups) launches fewer
// workgroups, which then take several pieces each and leave compute units free for other
// kernels.  How pieces are dealt to the 8 XCDs is piece_of_workgroup's business:

// Which part (tile or piece) of the chunk table workgroup b takes.  Workgroup b runs on XCD b % 8.  Within
// a block of 8 chunks' worth of workgroups, XCD k takes every part of chunk k, so that the parts' reads of
// the chunk's table entries and of shared 128-byte lines of a peer's codes meet in one L2 (compressed pass on
// 1 GiB buckets, N = 16: 1.150 ms against 1.25 in the plain order).  The last, incomplete block keeps the
// plain order.  A bijection on [0, num_pieces) for any grid size.
template <bool XCD, typename T>
__device__ __forceinline__ T piece_of_workgroup(T b, unsigned per_chunk, T num_pieces)
{
    if (!XCD) return b;
#if CDSGD_XCD_PIECES
    const T group = (T)8 * per_chunk;
    const T blk = b / group, within = b % group;
    if ((blk + 1) * group <= num_pieces) return (blk * 8 + within % 8) * per_chunk + within / 8;
#endif
    return b;
}

}  // namespace
