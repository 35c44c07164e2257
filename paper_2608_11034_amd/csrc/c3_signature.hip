// Streaming signature kernel of C3 for gfx950.
//
// Per (replica, chunk) it computes the C3SIG-1 signature -- a per-chunk
// reading of the paper's comparable evidence H_w(dtype, shape, bytes)
// (Sec. 5.2) -- and, in the same single pass over HBM, the chunk's NaN/Inf
// counts, absmax and fp64 sum / sum of squares of the finite elements.
//
// C3SIG-1 over a chunk of n bytes: the bytes, zero-padded to a multiple of 16,
// are little-endian u32 words m[0..D-1], D = 4 ceil(n / 16).  Keys K[i] are
// the low 32 bits of SplitMix64 outputs i = 0..257 from a fixed seed.  For
// each word pair p = 2i, with q = p mod 256 and beta = (p div 256) * 0x9E3779B9
// (all u32 arithmetic wraps):
//     A += (m[p] + K[q] + beta) * (m[p+1] + K[q+1] + beta)      (u64, wraps)
//     B += (m[p] + K[q+2] + beta) * (m[p+1] + K[q+3] + beta)
// which is the NH hash of UMAC with a Toeplitz-shifted second key row.  The
// signature is an fmix64 chain over (tag ^ dtype << 32 ^ ndim, shape dims,
// chunk index, n, A, B).  A and B are sums, so any partition of the chunk
// gives the same bits.
//
// Work decomposition: a chunk is cut into tiles of tile_bytes (whole KiB; the
// last tile of a chunk may be shorter).  A tile's 1 KiB blocks form four
// quarters, block b belonging to quarter b mod 4; every lane loads 16 bytes of
// a block with one 128-bit load, so one wave-wide load covers exactly 256
// words and lane l always owns key positions 4l .. 4l+5 (held in VGPRs for
// the whole kernel) while beta is wave-uniform.  Either a 256-thread workgroup
// folds a tile, one wave per quarter (signature_kernel), or one wave folds
// all four (signature_wave_kernel, small tiles in large numbers).  Lanes
// reduce with xor butterflies, quarters combine in a fixed order, and each
// tile writes one 64-byte partial.  When a chunk is a single tile the chunk
// record is written directly; otherwise a finalize kernel combines the
// chunk's partials in tile order.  The per-tile arithmetic depends neither on
// which workgroup or wave runs it nor on which of the two kernels does, so
// results are independent of the grid size, of the tile order and of what
// else is signed in the launch: large launches take their tiles through the
// XCD map (xcd_map_tile), the others in order.
//
// Non-finite screen: a lane sums its elements in fp64 without looking at
// them.  A non-finite element is the only way its sum or sum of squares can
// become non-finite (finite fp32/bf16/fp16 values cannot overflow fp64 here),
// so a lane whose sums end non-finite re-reads its own segments and
// classifies every element.  Healthy data never takes that path.
#include <string.h>

#include <type_traits>

#include "c3_device.h"
#include "c3_fold.h"
#include "c3_internal.h"
#include "c3_localize_block.h"
#include "c3_tail.h"
#include "c3_vote_row.h"

namespace c3 {

__device__ inline int find_segment(const int64_t* base, int n, int64_t j) {
    // largest t in [0, n) with base[t] <= j  (base[0] = 0, base ascending)
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (base[mid] <= j) lo = mid; else hi = mid;
    }
    return lo;
}

// find_segment by a whole wave: each round its lanes probe 64 evenly spaced
// entries of the range that holds the answer, so 121 tensors take two
// dependent loads instead of seven.  j is uniform; so is the result.
__device__ inline int find_segment_wave(const int64_t* base, int n, int64_t j, int lane) {
    int lo = 0;                       // base[lo] <= j
    while (n > 1) {
        const int step = (n + 63) >> 6;
        const int p = lane * step;
        const int k = __builtin_popcountll(ballot64(p < n && base[lo + p] <= j));   // a prefix, >= 1
        const int at = (k - 1) * step;
        n = n - at < step ? n - at : step;
        lo += at;
    }
    return lo;
}

// a / b, in 32 bits where a allows it (a 64-bit division is a sequence of
// more than a hundred instructions; the operands here are wave-uniform)
__device__ inline uint64_t udiv(uint64_t a, uint32_t b) {
    if (b == 1u) return a;
    if ((a >> 32) == 0ull) return (uint32_t)a / b;
    return a / b;
}

// The replica of tile i of a launch of gtiles tiles per replica.
__device__ inline int64_t replica_of(int64_t i, int64_t gtiles) {
    return ((i | gtiles) >> 32) == 0 ? (int64_t)((uint32_t)i / (uint32_t)gtiles) : i / gtiles;
}

// Where a kernel finds the plan: staged into the workspace, or, when it is
// small, among the kernel's own arguments, which saves the launch that stages
// it and the first trip to memory of every look-up (place_plan).
struct StagedPlan {
    const SigPlan* p;
    static constexpr bool kChunkTable = true;
    __device__ const SigPlan* plan() const { return p; }
    __device__ char* workspace() const {
        return const_cast<char*>(reinterpret_cast<const char*>(p));
    }
};
struct ArgPlan {
    alignas(16) unsigned char bytes[kArgPlanBytes];
    char* ws;
    static constexpr bool kChunkTable = false;      // the chunk-to-tensor table stays behind
    __device__ const SigPlan* plan() const { return reinterpret_cast<const SigPlan*>(bytes); }
    __device__ char* workspace() const { return ws; }
};

template <typename F>
static void with_plan(const PlanSource& src, const F& launch) {
    if (src.arg_bytes != 0) {
        ArgPlan a;
        memcpy(a.bytes, src.arg, src.arg_bytes);
        a.ws = static_cast<char*>(src.ws);
        launch(a);
    } else {
        launch(StagedPlan{static_cast<const SigPlan*>(src.ws)});
    }
}

// The plan's arrays, and where a tile's bytes are.
struct PlanView {
    const uint64_t* ptrs;
    const int64_t* tile_base;
    const int64_t* chunk_base;
    const int32_t* order;
    const int64_t* gtile;
    const TensorInfo* tinfo;
    TilePartial* partials;
    template <typename P>
    __device__ explicit PlanView(const P& src) {
        const SigPlan* plan = src.plan();
        const char* pb = reinterpret_cast<const char*>(plan);
        ptrs = reinterpret_cast<const uint64_t*>(pb + plan->off_ptrs);
        tile_base = reinterpret_cast<const int64_t*>(pb + plan->off_tile_base);
        chunk_base = reinterpret_cast<const int64_t*>(pb + plan->off_chunk_base);
        order = reinterpret_cast<const int32_t*>(pb + plan->off_order);
        gtile = reinterpret_cast<const int64_t*>(pb + plan->off_gtile);
        tinfo = reinterpret_cast<const TensorInfo*>(pb + plan->off_tmeta);
        partials = reinterpret_cast<TilePartial*>(src.workspace() + plan->off_partials);
    }
};

// Tile lt of a tensor of nbytes bytes: tile lt mod tpc of chunk lt / tpc.
struct TileSpan {
    uint64_t chunk, off;   // chunk within the tensor, first byte
    uint32_t len, blk0;    // bytes, first 1 KiB block within the chunk
};

__device__ inline TileSpan tile_span(uint64_t lt, uint32_t tpc, uint64_t chunk_bytes,
                                     uint64_t tile_bytes, uint64_t nbytes) {
    TileSpan s;
    s.chunk = udiv(lt, tpc);
    const uint64_t within = (lt - s.chunk * tpc) * tile_bytes;
    s.off = s.chunk * chunk_bytes + within;
    const uint64_t end = min(nbytes, (s.chunk + 1) * chunk_bytes);
    s.len = end > s.off ? (uint32_t)min(tile_bytes, end - s.off) : 0u;
    s.blk0 = (uint32_t)(within >> 10);
    return s;
}

// fold_lane for a compile-time type, or (kMixed) the tensor's own
constexpr int kMixed = -1;

template <int DT, int U, int NW, bool FOLD>
__device__ inline LaneFold<4 / NW> fold_tile(int dtype, const uint8_t* tile, uint32_t len, uint32_t blk0,
                                     const LaneKeys& K, int wave, int lane) {
    if constexpr (DT != kMixed) {
        return fold_lane<DT, U, NW, FOLD>(tile, len, blk0, K, wave, lane);
    } else {
        switch (__builtin_amdgcn_readfirstlane(dtype)) {
            case C3_F32: return fold_lane<C3_F32, U, NW, FOLD>(tile, len, blk0, K, wave, lane);
            case C3_BF16: return fold_lane<C3_BF16, U, NW, false>(tile, len, blk0, K, wave, lane);
            case C3_F16: return fold_lane<C3_F16, U, NW, false>(tile, len, blk0, K, wave, lane);
            default: return fold_lane<C3_RAW, U, NW, false>(tile, len, blk0, K, wave, lane);
        }
    }
}

// The plan lists the tensors grouped by element type (order[], stable in call
// order) with a tile prefix over that order (gtile[]); a launch covers group
// positions [gk0, gk1) of every replica: the one type present, or all of them
// with DT = kMixed.
//
// One workgroup per tile.
template <int DT, int U, bool FOLD, typename P>
__global__ void __launch_bounds__(kSigThreads, C3_SIG_WAVES_PER_EU)
    signature_kernel(const P src, c3_chunk_record_t* __restrict__ records, int gk0, int gk1,
                     int64_t gtiles, int mapped, uint32_t* clear) {
    if (clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0u;
    const SigPlan* const plan = src.plan();
    __shared__ TilePartial lds[kSigThreads / 64];
    const int lane = threadIdx.x & 63;
    // the wave index, uniform across the wave (keeps beta and addresses scalar)
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const PlanView pv(src);
    const int T = plan->T;
    const int64_t ntiles = gtiles * plan->R;
    const uint64_t tile_bytes = plan->tile_bytes, chunk_bytes = plan->chunk_bytes;
    const uint32_t tpc = plan->tiles_per_chunk;
    const int64_t g0 = pv.gtile[gk0];
    const LaneKeys K = lane_keys(lane);

    // a mapped launch: one tile per workgroup, from the XCD map; otherwise
    // tiles blockIdx.x, blockIdx.x + gridDim.x, ...
    for (int64_t i = mapped ? xcd_map_tile(blockIdx.x, ntiles) : (int64_t)blockIdx.x; i < ntiles;
         i += mapped ? ntiles : (int64_t)gridDim.x) {
        const int64_t r = replica_of(i, gtiles);
        const int64_t j = g0 + (i - r * gtiles);
        const int k = gk0 + find_segment_wave(pv.gtile + gk0, gk1 - gk0, j, lane);
        const int t = pv.order[k];
        const int64_t lt = j - pv.gtile[k];
        const TileSpan ts = tile_span((uint64_t)lt, tpc, chunk_bytes, tile_bytes, pv.tinfo[t].nbytes);
        const uint8_t* tile = reinterpret_cast<const uint8_t*>(pv.ptrs[r * T + t]) + ts.off;

        const LaneFold<1> f = fold_tile<DT, U, 4, FOLD>(pv.tinfo[t].dtype, tile, ts.len, ts.blk0,
                                                     K, wave, lane);
        const TilePartial wp = wave_reduce(f);
        if (lane == 0) lds[wave] = wp;
        __syncthreads();
        if (threadIdx.x == 0) {
            TilePartial p = lds[0];
#pragma unroll
            for (int w = 1; w < kSigThreads / 64; ++w) partial_add(p, lds[w]);
            if (plan->direct)  // one tile per chunk
                write_record(&records[r * plan->C + pv.chunk_base[t] + lt], pv.tinfo[t], t,
                             (uint64_t)lt, ts.len, p);
            else
                pv.partials[r * plan->tiles_per_replica + pv.tile_base[t] + lt] = p;
        }
        __syncthreads();
    }
}

// One wave per tile, `run` consecutive tiles (at most kWaveRunMax) per wave:
// tiles up to kWaveTileMax bytes.  A workgroup on a 16 KiB tile has four loads in
// flight per lane and then a barrier, four reductions and a record to write:
// its latency, not the memory, sets the pace (2.8 TB/s on 1.6 GB of bf16 in
// 16 KiB chunks).  A wave per tile keeps 16 loads in flight per lane; the
// keys and the look-ups serve the whole run, and the run's records are hashed
// and written by one lane each, together.  No barrier: waves are independent.
// Each quarter of a tile's blocks is summed apart, as the four waves of a
// workgroup do, so both kernels write the same bits.
struct RunTile {
    TilePartial p;
    int64_t r, lt;
    int32_t t;
    uint32_t len;
};

template <int DT, int U, bool FOLD, typename P>
__global__ void __launch_bounds__(kSigThreads, C3_SIG_WAVES_PER_EU)
    signature_wave_kernel(const P src, c3_chunk_record_t* __restrict__ records, int gk0, int gk1,
                          int64_t gtiles, int run, uint32_t* clear) {
    if (clear != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *clear = 0u;
    const SigPlan* const plan = src.plan();
    __shared__ RunTile done[kSigThreads / 64][kWaveRunMax];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t ntiles = gtiles * plan->R;
    const PlanView pv(src);
    const int T = plan->T;
    const uint64_t tile_bytes = plan->tile_bytes, chunk_bytes = plan->chunk_bytes;
    const uint32_t tpc = plan->tiles_per_chunk;
    const int64_t g0 = pv.gtile[gk0];
    const LaneKeys K = lane_keys(lane);
    const int64_t nruns = (ntiles + run - 1) / run;
    for (int64_t w = (int64_t)blockIdx.x * (kSigThreads / 64) + wave; w < nruns;
         w += (int64_t)gridDim.x * (kSigThreads / 64)) {
        const int64_t i0 = w * run;
        const int count = (int)min((int64_t)run, ntiles - i0);
        int64_t r = replica_of(i0, gtiles);
        int64_t j = g0 + (i0 - r * gtiles);
        int k = gk0 + find_segment_wave(pv.gtile + gk0, gk1 - gk0, j, lane);
        for (int m = 0; m < count; ++m, ++j) {
            if (j == g0 + gtiles) {                    // on to the next replica
                ++r;
                j = g0;
                k = gk0;
            }
            while (j >= pv.gtile[k + 1]) ++k;          // every tensor has a tile: at most one step
            const int t = pv.order[k];
            const int64_t lt = j - pv.gtile[k];
            const TileSpan ts =
                tile_span((uint64_t)lt, tpc, chunk_bytes, tile_bytes, pv.tinfo[t].nbytes);
            const uint8_t* tile = reinterpret_cast<const uint8_t*>(pv.ptrs[r * T + t]) + ts.off;
            const LaneFold<4> f =
                fold_tile<DT, U, 1, FOLD>(pv.tinfo[t].dtype, tile, ts.len, ts.blk0, K, 0, lane);
            const TilePartial p = wave_reduce(f);
            if (lane == 0) done[wave][m] = RunTile{p, r, lt, t, ts.len};
        }
        wave_lds_sync();
        if (lane < count) {
            const RunTile d = done[wave][lane];
            if (plan->direct)
                write_record(&records[d.r * plan->C + pv.chunk_base[d.t] + d.lt], pv.tinfo[d.t],
                             d.t, (uint64_t)d.lt, d.len, d.p);
            else
                pv.partials[d.r * plan->tiles_per_replica + pv.tile_base[d.t] + d.lt] = d.p;
        }
        wave_lds_sync();                               // read before the next run writes
    }
}

// Where chunk c of replica r has its tile partials, and what its record needs.
struct ChunkParts {
    const TilePartial* pp;
    int64_t nt;            // tiles
    uint64_t k, n;         // chunk within the tensor, bytes
    int t;
};

template <typename P>
__device__ inline ChunkParts chunk_parts(const P& src, int64_t r, int64_t c) {
    const SigPlan* const plan = src.plan();
    const char* pb = reinterpret_cast<const char*>(plan);
    const PlanView pv(src);
    ChunkParts o;
    if constexpr (P::kChunkTable)
        o.t = reinterpret_cast<const int32_t*>(pb + plan->off_chunk_tensor)[c];
    else
        o.t = find_segment(pv.chunk_base, plan->T, c);
    o.k = (uint64_t)(c - pv.chunk_base[o.t]);
    const uint64_t nbytes = pv.tinfo[o.t].nbytes;
    const int64_t tb = pv.tile_base[o.t];
    const int64_t tiles_t = pv.tile_base[o.t + 1] - tb;
    const int64_t lt0 = (int64_t)o.k * plan->tiles_per_chunk;
    o.nt = min((int64_t)plan->tiles_per_chunk, tiles_t - lt0);
    o.pp = pv.partials + r * plan->tiles_per_replica + tb + lt0;
    const uint64_t coff = o.k * plan->chunk_bytes;
    o.n = nbytes > coff ? min(plan->chunk_bytes, nbytes - coff) : 0;
    return o;
}

// Record of (replica r, chunk c) by one thread, where a chunk has at most
// kThreadCombine tiles.
template <typename P>
__device__ inline void combine_chunk(const P& src, int64_t r, int64_t c, c3_chunk_record_t* out) {
    const ChunkParts cp = chunk_parts(src, r, c);
    const TilePartial p = combine_few(cp.pp, (int)cp.nt);
    write_record(out, PlanView(src).tinfo[cp.t], cp.t, cp.k, cp.n, p);
}

// Combine the partials of each (replica, chunk), sixteen lanes each.
template <typename P>
__global__ void __launch_bounds__(256) finalize_kernel(const P src,
                                                       c3_chunk_record_t* __restrict__ records) {
    const SigPlan* const plan = src.plan();
    const int64_t C = plan->C;
    const int64_t total = C * plan->R;
    const int l = threadIdx.x & 15;
    for (int64_t idx = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4); idx < total;
         idx += (int64_t)gridDim.x * 16) {
        const int64_t r = idx / C;
        const ChunkParts cp = chunk_parts(src, r, idx - r * C);
        const TilePartial p = combine_row(cp.pp, cp.nt, l);
        if (l == 0) write_record(&records[idx], PlanView(src).tinfo[cp.t], cp.t, cp.k, cp.n, p);
    }
}

// ---------------------------------------------------------------------------
// Records, votes and lists of a small plan in one workgroup (c3_tail.h), in
// place of three launches of a few microseconds each: plans of up to
// kTailMaxChunks chunks and kTailMaxRecords records.  `mode` says where the
// records are: kTailReady as the streaming or the finalize kernel wrote them,
// else combined here from tile partials, by a thread or by sixteen lanes each.
// ---------------------------------------------------------------------------
enum { kTailReady = 0, kTailThread = 1, kTailRow = 2 };

template <typename P>
__global__ void __launch_bounds__(kTailThreads) small_tail_kernel(
    const P src, c3_chunk_record_t* __restrict__ records, int mode, TailOut out) {
    const SigPlan* const plan = src.plan();
    __shared__ c3_chunk_record_t rec[kTailMaxRecords];
    const int R = plan->R;
    const int C = (int)plan->C;
    if (mode == kTailRow) {
        const int l = threadIdx.x & 15;
        for (int i = threadIdx.x >> 4; i < R * C; i += kTailThreads / 16) {
            const ChunkParts cp = chunk_parts(src, i / C, i % C);
            const TilePartial p = combine_row(cp.pp, cp.nt, l);
            if (l == 0) {
                write_record(&rec[i], PlanView(src).tinfo[cp.t], cp.t, cp.k, cp.n, p);
                records[i] = rec[i];
            }
        }
    } else {
        for (int i = threadIdx.x; i < R * C; i += kTailThreads) {
            if (mode == kTailReady) {
                rec[i] = records[i];
            } else {
                combine_chunk(src, i / C, i % C, &rec[i]);
                records[i] = rec[i];
            }
        }
    }
    tail_votes_and_lists(rec, R, C, out);
}

bool small_tail_fits(int R, int64_t C) {
    return C >= 1 && C <= kTailMaxChunks && R * C <= kTailMaxRecords;
}

hipError_t launch_small_tail(const PlanSource& src, const SigPlan& hplan, c3_chunk_record_t* records,
                             bool ready, const TailOut& out, hipStream_t stream) {
    const int mode = ready ? kTailReady
                     : hplan.tiles_per_chunk <= (uint32_t)kThreadCombine ? kTailThread : kTailRow;
    with_plan(src, [&](const auto& p) {
        using P = std::decay_t<decltype(p)>;
        hipLaunchKernelGGL(small_tail_kernel<P>, dim3(1), dim3(kTailThreads), 0, stream, p, records,
                           mode, out);
    });
    return hipGetLastError();
}

// Records that the finalize kernel should combine before the tail: more than
// a thread combines, and for the one-workgroup tail more than a few rounds of
// its groups of sixteen lanes.
bool finalize_first(const SigPlan& hplan, bool small) {
    if (hplan.direct || hplan.tiles_per_chunk <= (uint32_t)kThreadCombine) return false;
    return !small || hplan.C * hplan.R > 4 * (kTailThreads / 16);
}

// ---------------------------------------------------------------------------
// Tail of c3_check: the records of every (replica, chunk) from their tile
// partials (at most kThreadCombine a chunk) or as the streaming or finalize
// kernel wrote them (`ready`), the exact vote of every chunk (exact_vote_row,
// the rule of c3_consensus) and the lists of c3_localize, in one launch:
//   - a workgroup of kCheckThreads threads takes CPB = kCheckThreads / N
//     consecutive chunks (a segment), one thread per (chunk, replica slot),
//     so the R records of a chunk are combined in parallel and meet in LDS;
//   - one thread per chunk votes;
//   - with a staging area, the first wave scans the segment's outlier and
//     undecided counts (CPB <= 64 units: one wave) and writes the segment's
//     entries, summaries taken from the records in LDS, into the segment's
//     slots of the staging area, with the three counts in one word;
//   - the workgroup that arrives last scans the segments' counts in segment
//     order and copies every staged entry to its place in the caller's lists.
//     Segments are in chunk order and entries in (chunk, replica) order inside
//     a segment, so the lists come out in c3_localize's order.
// The handoff passes the staging area only, a few KiB, so it goes through
// agent-scope accesses, which meet where all XCDs look, and a wait for them
// before the arrival is counted; an agent-scope release would write back the
// XCD's whole L2, once per workgroup (17.9 us for the tail against 14 for two
// launches when that was tried).  The counter is cleared by the streaming
// kernel of the same call.
// ---------------------------------------------------------------------------
constexpr int kCheckThreads = 256;
constexpr int kCheckMaxListUnits = 8192;   // chunks whose lists go through the staging area
constexpr int kCheckMaxSegments = kCheckMaxListUnits / (kCheckThreads / 32);
// per step of 64 segments: outliers < 64 * CPB * N / 2 = 64 * kCheckThreads / 2,
// units <= 64 * 64
static_assert(64ll * kCheckThreads / 2 < (1ll << 24) && 64 * 64 < (1 << 20), "packed counts");

struct CheckStage {
    uint64_t* seg;            // [n_seg]: outliers (24 bits), undecided and attributed units (20 each)
    uint32_t* done;           // workgroups that have staged their segment
    c3_outlier_t* out;        // [n_seg][out_per_seg]
    int64_t* und;             // [n_seg][CPB]
    int32_t out_per_seg;
    int32_t cpb;
};
struct CheckLists {
    c3_outlier_t* outliers;
    int64_t out_cap;
    int64_t* undecided;
    int64_t und_cap;
    int64_t* counts;
};

__device__ __forceinline__ void agent_store(void* p, uint64_t v) {
    __hip_atomic_store(static_cast<uint64_t*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t agent_load(const void* p) {
    return __hip_atomic_load(static_cast<const uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
constexpr int kOutlierWords = sizeof(c3_outlier_t) / 8;
static_assert(sizeof(c3_outlier_t) % 8 == 0, "entries are copied in words");

// The lists from the staged segments, by one workgroup.  seg_word, off_o and
// off_u: kCheckMaxSegments entries each in LDS.
__device__ inline void place_lists(const CheckStage& stage, int n_seg, const CheckLists& lists,
                                   uint64_t* seg_word, int32_t* off_o, int32_t* off_u) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (wave == 0) {
        // segment offsets in segment order: one wave, 64 segments per step
        int64_t carry_o = 0, carry_u = 0, carry_a = 0;
        for (int base = 0; base < n_seg; base += 64) {
            const int sgi = base + lane;
            const uint64_t packed = sgi < n_seg ? agent_load(&stage.seg[sgi]) : 0ull;
            const uint64_t incl = wave_inclusive_scan(packed, lane);
            const uint64_t excl = incl - packed;
            if (sgi < n_seg) {
                seg_word[sgi] = packed;
                off_o[sgi] = (int32_t)(carry_o + (int64_t)(excl & 0xFFFFFFull));
                off_u[sgi] = (int32_t)(carry_u + (int64_t)((excl >> 24) & 0xFFFFFull));
            }
            const uint64_t tot = shfl_u64(incl, 63);
            carry_o += (int64_t)(tot & 0xFFFFFFull);
            carry_u += (int64_t)((tot >> 24) & 0xFFFFFull);
            carry_a += (int64_t)((tot >> 44) & 0xFFFFFull);
        }
        if (lane == 0) {
            lists.counts[0] = carry_o;
            lists.counts[1] = carry_u;
            lists.counts[2] = carry_a;
        }
    }
    __syncthreads();
    for (int sgi = wave; sgi < n_seg; sgi += kCheckThreads / 64) {
        const int n_o = (int)(seg_word[sgi] & 0xFFFFFFull), n_u = (int)((seg_word[sgi] >> 24) & 0xFFFFFull);
        const c3_outlier_t* so = stage.out + (int64_t)sgi * stage.out_per_seg;
        for (int j = lane; j < n_o; j += 64) {
            const int64_t d = (int64_t)off_o[sgi] + j;
            if (d >= lists.out_cap) continue;
            uint64_t w[kOutlierWords];
#pragma unroll
            for (int i = 0; i < kOutlierWords; ++i)
                w[i] = agent_load(reinterpret_cast<const uint64_t*>(&so[j]) + i);
#pragma unroll
            for (int i = 0; i < kOutlierWords; ++i) reinterpret_cast<uint64_t*>(&lists.outliers[d])[i] = w[i];
        }
        for (int j = lane; j < n_u; j += 64) {
            const int64_t d = (int64_t)off_u[sgi] + j;
            if (d < lists.und_cap)
                lists.undecided[d] = (int64_t)agent_load(&stage.und[(int64_t)sgi * stage.cpb + j]);
        }
    }
}

template <int N, typename P>
__global__ void __launch_bounds__(kCheckThreads) check_vote_kernel(
    const P src, c3_chunk_record_t* __restrict__ records,
    bool ready, uint8_t* __restrict__ status, uint64_t* __restrict__ bitmap,
    int32_t* __restrict__ majority, CheckStage stage, CheckLists lists) {
    constexpr int CPB = kCheckThreads / N;
    static_assert(CPB <= 64, "a segment's units must fit one wave");
    // the records; after them, in the last workgroup, the segments' counts
    // and offsets
    __shared__ __align__(16) unsigned char shared[CPB * N * sizeof(c3_chunk_record_t)];
    static_assert(sizeof(shared) >= kCheckMaxSegments * 16, "segment tables");
    c3_chunk_record_t(*rec)[N] = reinterpret_cast<c3_chunk_record_t(*)[N]>(shared);
    __shared__ UnitVote votes[CPB];
    __shared__ uint32_t arrived;
    const SigPlan* const plan = src.plan();
    const int R = plan->R;
    const int64_t C = plan->C;
    const int slot = threadIdx.x % N;
    const int cu = threadIdx.x / N;
    const int64_t c = (int64_t)blockIdx.x * CPB + cu;
    if (slot < R && c < C) {
        c3_chunk_record_t* dst = &records[(int64_t)slot * C + c];
        if (ready) {
            rec[cu][slot] = *dst;
        } else {
            c3_chunk_record_t r;
            combine_chunk(src, slot, c, &r);
            *dst = r;
            rec[cu][slot] = r;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < CPB) {
        const int64_t u = (int64_t)blockIdx.x * CPB + threadIdx.x;
        if (u < C) {
            uint64_t e[N];
#pragma unroll
            for (int r = 0; r < N; ++r) e[r] = r < R ? rec[threadIdx.x][r].sig : 0ull;
            const UnitVote v = exact_vote_row<N>(e, R);
            status[u] = v.status;
            bitmap[u] = v.bitmap;
            majority[u] = v.majority;
            votes[threadIdx.x] = v;
        }
    }
    if (stage.seg == nullptr) return;
    __syncthreads();
    if (threadIdx.x < 64) {
        // this segment's entries, in (chunk, replica) order, into its slots
        const int lane = threadIdx.x;
        const int64_t u = (int64_t)blockIdx.x * CPB + lane;
        const bool valid = lane < CPB && u < C;
        UnitVote v{0ull, -1, (uint8_t)C3_AGREE};
        if (valid) v = votes[lane];
        const uint64_t n_o =
            valid && v.status != C3_INCONCLUSIVE ? (uint64_t)__builtin_popcountll(v.bitmap) : 0ull;
        const uint64_t n_u = valid && v.status == C3_INCONCLUSIVE ? 1ull : 0ull;
        const uint64_t packed = n_o | (n_u << 24) | ((uint64_t)(n_o != 0ull) << 44);
        const uint64_t incl = wave_inclusive_scan(packed, lane);
        const uint64_t excl = incl - packed;
        uint64_t po = excl & 0xFFFFFFull;
        const uint64_t pu = (excl >> 24) & 0xFFFFFull;
        c3_outlier_t* so = stage.out + (int64_t)blockIdx.x * stage.out_per_seg;
        for (uint64_t b = n_o ? v.bitmap : 0ull; b != 0ull; b &= b - 1ull, ++po) {
            const int r = __builtin_ctzll(b);
            union {
                c3_outlier_t o;
                uint64_t w[kOutlierWords];
            } e;
            outlier_from(e.o, u, r, v.majority, rec[lane][r], rec[lane][v.majority]);
#pragma unroll
            for (int i = 0; i < kOutlierWords; ++i)
                agent_store(reinterpret_cast<uint64_t*>(&so[po]) + i, e.w[i]);
        }
        if (n_u) agent_store(&stage.und[(int64_t)blockIdx.x * CPB + (int64_t)pu], (uint64_t)u);
        if (lane == 63) agent_store(&stage.seg[blockIdx.x], incl);
        // every staged store of this wave has reached the point where all
        // XCDs see it before the workgroup counts itself in
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if (lane == 0)
            arrived = __hip_atomic_fetch_add(stage.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (arrived != gridDim.x - 1) return;              // the whole workgroup leaves together
    asm volatile("" ::: "memory");
    uint64_t* seg_word = reinterpret_cast<uint64_t*>(shared);
    int32_t* off = reinterpret_cast<int32_t*>(seg_word + kCheckMaxSegments);
    place_lists(stage, (int)gridDim.x, lists, seg_word, off, off + kCheckMaxSegments);
}

int check_group_bound(int R) { return R <= 4 ? 4 : R <= 8 ? 8 : R <= 16 ? 16 : R <= 32 ? 32 : 0; }

// Staging bytes for the fused lists of C chunks at group bound N (0 when
// the tail leaves the lists to a separate localization).
static uint64_t check_stage_parts(int N, int64_t C, uint64_t& cnt_b, uint64_t& out_b,
                                  uint64_t& und_b, int& out_per_seg) {
    const int64_t cpb = kCheckThreads / N;
    const int64_t n_seg = (C + cpb - 1) / cpb;
    // a strict majority holds more than R / 2 replicas, so a chunk has at
    // most ceil(R / 2) - 1 < N / 2 outliers
    out_per_seg = (int)(cpb * (N / 2));
    cnt_b = (uint64_t)n_seg * 16;
    out_b = (uint64_t)n_seg * out_per_seg * sizeof(c3_outlier_t);
    und_b = (uint64_t)n_seg * cpb * 8;
    return ((cnt_b + 255) / 256 + (out_b + 255) / 256 + (und_b + 255) / 256) * 256;
}

uint64_t check_stage_bytes(int R, int64_t C) {
    const int N = check_group_bound(R);
    if (N == 0 || C > kCheckMaxListUnits) return 0;
    uint64_t a, b, c;
    int o;
    return check_stage_parts(N, C, a, b, c, o);
}

// The arrival counter, after the segments' words (16 bytes are kept a segment).
uint32_t* check_arrivals(int R, int64_t C, void* stage_ws) {
    const int64_t cpb = kCheckThreads / check_group_bound(R);
    const int64_t n_seg = (C + cpb - 1) / cpb;
    return reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(stage_ws) + 8 * n_seg);
}

hipError_t launch_check_tail(const PlanSource& src, const SigPlan& hplan, c3_chunk_record_t* records,
                             bool ready, uint8_t* status, uint64_t* bitmap, int32_t* majority,
                             c3_outlier_t* outliers, int64_t out_cap, int64_t* undecided,
                             int64_t und_cap, int64_t* counts, void* stage_ws,
                             hipStream_t stream) {
    const int N = check_group_bound(hplan.R);
    if (N == 0 || hplan.C <= 0) return hipErrorInvalidValue;
    const int64_t cpb = kCheckThreads / N;
    const int64_t blocks = (hplan.C + cpb - 1) / cpb;
    if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
    CheckStage st{nullptr, nullptr, nullptr, nullptr, 0, (int32_t)cpb};
    const CheckLists lists{outliers, out_cap, undecided, und_cap, counts};
    if (stage_ws != nullptr) {
        if (hplan.C > kCheckMaxListUnits) return hipErrorInvalidValue;
        uint64_t cnt_b, out_b, und_b;
        check_stage_parts(N, hplan.C, cnt_b, out_b, und_b, st.out_per_seg);
        unsigned char* w = static_cast<unsigned char*>(stage_ws);
        st.seg = reinterpret_cast<uint64_t*>(w);
        st.done = check_arrivals(hplan.R, hplan.C, stage_ws);
        w += (cnt_b + 255) / 256 * 256;
        st.out = reinterpret_cast<c3_outlier_t*>(w);
        w += (out_b + 255) / 256 * 256;
        st.und = reinterpret_cast<int64_t*>(w);
    }
    with_plan(src, [&](const auto& p) {
        using P = std::decay_t<decltype(p)>;
        auto vote = [&](auto n) {
            hipLaunchKernelGGL((check_vote_kernel<decltype(n)::value, P>), dim3((unsigned)blocks),
                               dim3(kCheckThreads), 0, stream, p, records, ready, status, bitmap,
                               majority, st, lists);
        };
        switch (N) {
            case 4: vote(std::integral_constant<int, 4>{}); break;
            case 8: vote(std::integral_constant<int, 8>{}); break;
            case 16: vote(std::integral_constant<int, 16>{}); break;
            default: vote(std::integral_constant<int, 32>{}); break;
        }
    });
    return hipGetLastError();
}

// Copies the staged plan from pinned host memory into the workspace on the
// compute queue (no copy engine, so no cross-engine synchronization): up to
// kFetchBlocks workgroups, four 16-byte loads per thread in flight, so a plan
// of up to 128 KiB is one round trip over the host link.  With `seen`, thread
// 0 of workgroup b then stores `seq` into seen[b] (system scope, pinned
// coherent host memory): every load of that workgroup has completed, since
// each thread stored what it loaded before the barrier, so the host may
// reuse the slot once every used word reads `seq`.
constexpr int kFetchThreads = 256;
constexpr int kFetchLoads = 4;

__global__ void __launch_bounds__(kFetchThreads) plan_fetch_kernel(const u32x4* __restrict__ src,
                                                                   u32x4* __restrict__ dst,
                                                                   int64_t n16, uint64_t* seen,
                                                                   uint64_t seq) {
    const int64_t stride = (int64_t)gridDim.x * kFetchThreads;
    for (int64_t i0 = (int64_t)blockIdx.x * kFetchThreads + threadIdx.x; i0 < n16;
         i0 += stride * kFetchLoads) {
        u32x4 v[kFetchLoads];
#pragma unroll
        for (int k = 0; k < kFetchLoads; ++k) {
            const int64_t i = i0 + (int64_t)k * stride;
            if (i < n16) v[k] = src[i];
        }
#pragma unroll
        for (int k = 0; k < kFetchLoads; ++k) {
            const int64_t i = i0 + (int64_t)k * stride;
            if (i < n16) dst[i] = v[k];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && seen != nullptr)
        __hip_atomic_store(seen + blockIdx.x, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

int plan_fetch_blocks(size_t bytes) {
    const int64_t n16 = (int64_t)((bytes + 15) / 16);
    const int64_t per = (int64_t)kFetchThreads * kFetchLoads;
    const int64_t b = (n16 + per - 1) / per;
    return b < 1 ? 1 : b > kFetchBlocks ? kFetchBlocks : (int)b;
}

hipError_t launch_plan_fetch(const void* host_src, void* dst, size_t bytes, hipStream_t stream,
                             uint64_t* seen, uint64_t seq) {
    const int64_t n16 = (int64_t)((bytes + 15) / 16);
    if (n16 == 0 && seen == nullptr) return hipSuccess;
    hipLaunchKernelGGL(plan_fetch_kernel, dim3((unsigned)plan_fetch_blocks(bytes)),
                       dim3(kFetchThreads), 0, stream, static_cast<const u32x4*>(host_src),
                       static_cast<u32x4*>(dst), n16, seen, seq);
    return hipGetLastError();
}

// A wave per tile instead of a workgroup: for small tiles, once there are
// enough of them that waves fill the chip.  Either way the results are the
// same bits.  Kernel us, workgroup / wave, bf16 (fp32 alike unless given):
//   16 KiB tiles   490: 9.4 / 9.2   1,954: 15.0 / 11.2   7,814: 46 / 28   97,658: 535 / 249
//   32 KiB tiles   246: 9.0 / 9.5     978: 11.5 / 10.7   7,814: 60 / 46   48,830: 332 / 241
//   48 KiB tiles   652: 11.3 / 12.0 1,304: 18.3 / 19.3   2,606: 28.9 / 27.1  32,554: 281 / 235
//   64 KiB tiles 3,908: 45.4 / 46.8 9,156: 98.6 / 95.4  24,416: 251 / 239 (fp32: 233 / 236)
//   96 KiB tiles 16,278: 238 / 240
// A lane that meets a NaN classifies its column of the tile, a quarter of it
// per wave in a workgroup and all of it in a wave: 490 tiles of 16 KiB with
// one NaN take 9.2 / 12.1 us, hence not below 1,024 tiles.
static bool wave_tiles(int dt, uint64_t tile_bytes, int64_t ntiles) {
    if (tile_bytes <= 32 * 1024) return ntiles >= 1024;
    if (tile_bytes <= 48 * 1024) return ntiles >= 2048;
    return dt != C3_F32 && tile_bytes <= kWaveTileMax && ntiles >= 8192;
}

template <int DT, bool FOLD>
static hipError_t launch_group(const PlanSource& src, c3_chunk_record_t* records, int gk0, int gk1,
                               int64_t gtiles, int R, uint64_t tile_bytes, int grid_blocks,
                               uint32_t* clear, hipStream_t stream) {
    const int64_t ntiles = gtiles * R;
    if (ntiles <= 0) return hipSuccess;
    if (wave_tiles(DT, tile_bytes, ntiles)) {
        // a run of kWaveRunBytes, shorter while the launch has fewer waves
        // than the chip holds at a time; results do not depend on it
        int64_t run = (int64_t)(kWaveRunBytes / tile_bytes);
        const int64_t fill = ntiles / kWaveFill;
        run = run > fill ? fill : run;
        run = run < 1 ? 1 : run > kWaveRunMax ? kWaveRunMax : run;
        const int64_t per = run * (kSigThreads / 64);
        int64_t grid = (ntiles + per - 1) / per;
        if (grid_blocks > 0 && grid > grid_blocks) grid = grid_blocks;
        if (grid > 0x7FFFFFFF) grid = 0x7FFFFFFF;
        with_plan(src, [&](const auto& p) {
            using P = std::decay_t<decltype(p)>;
            hipLaunchKernelGGL((signature_wave_kernel<DT, kUnroll, FOLD, P>), dim3((unsigned)grid),
                               dim3(kSigThreads), 0, stream, p, records, gk0, gk1, gtiles, (int)run, clear);
        });
        return hipGetLastError();
    }
    int64_t grid = grid_blocks > 0 ? grid_blocks : ntiles;
    if (grid > ntiles) grid = ntiles;
    const int mapped = grid_blocks <= 0 && xcd_map_applies(ntiles, tile_bytes);
    if (mapped) grid = xcd_map_grid(ntiles);
    if (grid > 0x7FFFFFFF) grid = 0x7FFFFFFF;
    with_plan(src, [&](const auto& p) {
        using P = std::decay_t<decltype(p)>;
        hipLaunchKernelGGL((signature_kernel<DT, kUnroll, FOLD, P>), dim3((unsigned)grid), dim3(kSigThreads),
                           0, stream, p, records, gk0, gk1, gtiles, mapped, clear);
    });
    return hipGetLastError();
}

hipError_t launch_signature(const PlanSource& src, const SigPlan& hplan, const SigGroups& groups,
                            c3_chunk_record_t* records, int grid_blocks, bool finalize,
                            uint32_t* clear, hipStream_t stream, hipEvent_t ev0, hipEvent_t ev1) {
    hipError_t e;
    if (ev0 && (e = hipEventRecord(ev0, stream)) != hipSuccess) return e;
    int only = -1, types = 0;
    for (int d = 0; d < 4; ++d)
        if (groups.k1[d] > groups.k0[d]) {
            only = d;
            ++types;
        }
    auto launch = [&](auto dt, auto fold) {
        constexpr int DT = decltype(dt)::value;
        constexpr bool FOLD = decltype(fold)::value;
        const int gk0 = DT == kMixed ? 0 : groups.k0[only], gk1 = DT == kMixed ? hplan.T : groups.k1[only];
        const int64_t gt = DT == kMixed ? hplan.tiles_per_replica : groups.tiles[only];
        return launch_group<DT, FOLD>(src, records, gk0, gk1, gt, hplan.R, hplan.tile_bytes, grid_blocks,
                                clear, stream);
    };
    // several types in one launch: a launch for each drains the chip between
    // them.  us per check of bf16 matrices with fp32 norms and fp16 biases, a
    // launch per type / one: 0.04 GB 33.1 / 16.1, 1.1 GB in 96 KiB tiles 203.9 /
    // 189.5, 8.6 GB in 128 KiB tiles 1,279 / 1,260, 4.3 and 17.2 GB in 256 KiB
    // tiles 634 / 618 and 2,418 / 2,414
    using std::integral_constant;
    const bool f = hplan.folds != 0;           // of fp32 tensors only
    if (types > 1)
        e = f ? launch(integral_constant<int, kMixed>{}, std::true_type{})
              : launch(integral_constant<int, kMixed>{}, std::false_type{});
    else if (only == C3_F32)
        e = f ? launch(integral_constant<int, C3_F32>{}, std::true_type{})
              : launch(integral_constant<int, C3_F32>{}, std::false_type{});
    else if (only == C3_BF16) e = launch(integral_constant<int, C3_BF16>{}, std::false_type{});
    else if (only == C3_F16) e = launch(integral_constant<int, C3_F16>{}, std::false_type{});
    else e = launch(integral_constant<int, C3_RAW>{}, std::false_type{});
    if (e != hipSuccess) return e;
    if (ev1 && (e = hipEventRecord(ev1, stream)) != hipSuccess) return e;
    if (!hplan.direct && finalize) {
        const int64_t total = hplan.C * hplan.R;
        const int64_t blocks = (total + 15) / 16 < 65536 ? (total + 15) / 16 : 65536;
        with_plan(src, [&](const auto& p) {
            using P = std::decay_t<decltype(p)>;
            hipLaunchKernelGGL(finalize_kernel<P>, dim3((unsigned)blocks), dim3(256), 0, stream, p,
                               records);
        });
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace c3
