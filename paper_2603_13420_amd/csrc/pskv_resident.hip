// Resident-prefix MFMA kernels of batched candidate-suffix attention for gfx950
// (bf16 tensors, head dim 128, prefix of at most 256 rows).
//
// One persistent workgroup per compute unit owns one KV head.  It copies that head's whole
// prefix K and V (the compact prefix cache of Sec. 4.2: one copy, never expanded over the
// candidates) into LDS once, and then its 8 wavefronts walk independently, without any
// further workgroup barrier, over 32-row blocks of the stacked query rows
//     r = (b*S + i)*G + g      (suffix-centric alignment, Sec. 4.3)
// of that head.  For each block a wavefront runs Eq. 2 over [prefix ; own suffix] with one
// online-softmax state per row: prefix tiles of 32 keys come from LDS, the candidate's own
// suffix K rows come straight from global memory and its V rows through a 4 KB per-wave
// scratch tile.
//
// Two kernels share this layout.  The general one handles any shape.  The pipelined one
// handles the common case in which every 32-row block lies inside one candidate (because the
// candidates' rows fill whole blocks, or nearly, each then taking blocks of its own) and the
// suffix fits one 32-key step: it overlaps, inside each wavefront, the score product of the
// next tile (matrix cores) with the exponentials of the current one (vector ALU), requests
// everything it needs from global memory a full block ahead, and never branches on data.
// The third takes calls that bring suffix lengths, S <= 32 and 1 <= P, whatever their candidates' rows fill, where 32-bit and 24-bit
// offsets reach (packed_args): the same pipeline over packed rows, valid ones only (pskv_packed.hpp).
// Operand layouts and the pieces shared with the streaming kernels are in pskv_mfma.hpp.
#include "pskv_packed.hpp"

namespace pskv {
namespace {

constexpr int kMaxTiles = 8; // resident prefix: at most 256 keys

// Copies the prefix K/V of the current virtual head into the fragment-major LDS images (whole
// workgroup of 512 threads).  All global loads are issued before the first LDS write, so their
// latencies overlap.
__device__ inline void stage_prefix(const Args &a, const Ctx &X, int ntiles, lds_u8 *kimg, lds_u8 *vimg, int tid)
{
    // The thread's place in the images is worked out here, from a thread id the compiler cannot
    // trace back, and the staging registers are defined on every path: kept alive across the
    // block loops of the callers instead, these values would be spilled.
    asm volatile("" : "+v"(tid));
    const TileSlot t = make_tile_slot(tid);
    uintx4 kv[kMaxTiles] = {}, vv[kMaxTiles] = {};
#pragma unroll
    for (int kt = 0; kt < kMaxTiles; ++kt)
        if (kt < ntiles)
            load_tile_chunks(a, X, t, kt, kv[kt], vv[kt]);
#pragma unroll
    for (int kt = 0; kt < kMaxTiles; ++kt)
        if (kt < ntiles)
            write_tile_chunks(X, t, kt, kimg + kt * kTileBytes, vimg + kt * kTileBytes, tid, kv[kt], vv[kt]);
}

// max_tiles: tiles of the padded prefix length; it fixes the LDS layout for every instruction.
__device__ inline Ctx make_ctx(const Args &a, lds_u8 *smem, int max_tiles, int tid)
{
    Ctx X;
    X.lane = tid & 63;
    X.h = X.lane >> 5;
    X.c32 = X.lane & 31;
    X.Mtot = a.C * a.S * a.G;
    X.c = a.scale * kLog2e;
    X.k_lane = smem + X.lane * 16;
    X.v_lane = smem + max_tiles * kTileBytes + X.lane * 8;
    X.scr = smem + 2 * max_tiles * kTileBytes + __builtin_amdgcn_readfirstlane(tid >> 6) * kScrBytes;
    X.sv_row_lo = 4 * ((X.c32 >> 4) & 1) + ((X.c32 >> 1) & 3);
    X.sv_chunk_lo = 2 * ((X.c32 >> 3) & 1) + (X.c32 & 1);
    return X;
}

// ------------------------------------------------------------------------------------------
// General path: one block, start to finish, nothing in flight across blocks.  Any shape:
// several candidates per block, suffixes longer than one step, no prefix at all.
// ------------------------------------------------------------------------------------------
__device__ __attribute__((always_inline)) void general_block(const Args &a, const Ctx &X, int ntiles, int blk)
{
    const int r0 = blk * kBlockRows;
    const Row row = decode_row(a, X, blk);
    const bool rvalid = row.rin && (int)row.ri < clamp_len(a, row.rlen);
    if (__builtin_amdgcn_ballot_w64(rvalid) == 0) {
        store_zero_block(a, X, r0, row);
        return;
    }
    uintx4 q[8];
    load_q(a, X, row, q);

    RowState st;
    st.m = -INFINITY;
    st.l = 0.f;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            st.o[dt][e] = 0.f;

    for (int kt = 0; kt < ntiles; ++kt) // prefix part: every row sees every real prefix key
        prefix_tile_classic(X, X.k_lane + kt * kTileBytes, X.v_lane + kt * kTileBytes, X.P - kt * kTileKeys, q, st);
    suffix_classic(a, X, r0, row, q, st);
    store_block(a, X, r0, row, rvalid, st.m, st.l, st.o);
}

// Work distribution shared by both kernels.  A "virtual head" is one (instruction, KV head)
// pair; there are VH = Np*Hkv of them, each with its own prefix and its own C*S*G stacked
// rows.  The grid is per_vh * vh_slots workgroups: workgroup w serves virtual heads
// w % vh_slots, + vh_slots, ... (consecutive workgroup ids, one per XCD in turn, take
// consecutive KV heads) and, within each, a share w / vh_slots out of per_vh of the row blocks.
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void resident_general_kernel(Args a, int per_vh, int vh_slots, int max_tiles)
{
    extern __shared__ __align__(16) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    Ctx X = make_ctx(a, smem, max_tiles, tid);
    const int nblocks = (X.Mtot + kBlockRows - 1) / kBlockRows;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int VH = a.Np * a.Hkv;
    for (int vh = blockIdx.x % vh_slots; vh < VH; vh += vh_slots) {
        set_vhead(a, X, vh);
        const int ntiles = (X.P + kTileKeys - 1) / kTileKeys;
        __syncthreads(); // every wavefront is done with the images of the virtual head before
        stage_prefix(a, X, ntiles, smem, smem + max_tiles * kTileBytes, tid);
        __syncthreads();
        for (int blk = (blockIdx.x / vh_slots) * kNW + wave; blk < nblocks; blk += per_vh * kNW)
            general_block(a, X, ntiles, blk);
    }
}

// ------------------------------------------------------------------------------------------
// Pipelined path.  Preconditions (checked by the launcher): every 32-row block lies inside one
// candidate; S <= 32, so the suffix is one 32-key step; and the prefix has at least three tiles.
//
// Softmax without per-tile maxima: the first prefix tile fixes the row's reference maximum;
// later tiles take exp2 relative to it whatever their own maximum is (a larger score just gives
// a weight above one, which fp32 sums and bf16 weights hold at full relative precision).  If a
// row's sum ends up at or above kBig, the wavefront goes over all its blocks once more with
// the general path after its main loop (rare; kept out of the main loop so that it costs it no
// registers).
// ------------------------------------------------------------------------------------------
// WHOLE: S*G is a multiple of 32, the blocks are those of the stacked rows.  Otherwise a candidate has
// nb blocks of its own, the last one being what is left (its rows past the candidate's stand in for the
// last one and are not stored).
template <bool WHOLE>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void resident_pipelined_kernel(Args a, int per_vh, int vh_slots, int max_tiles, int nb, FastDiv div_nb)
{
    extern __shared__ __align__(16) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    Ctx X = make_ctx(a, smem, max_tiles, tid);
    const int rows_c = a.S * a.G; // rows of a candidate
    const int nblocks = WHOLE ? (X.Mtot + kBlockRows - 1) / kBlockRows : a.C * nb;
    const int VH = a.Np * a.Hkv;
    auto kimg = [&](int t) { return X.k_lane + t * kTileBytes; };
    auto vimg = [&](int t) { return X.v_lane + t * kTileBytes; };

    // Candidate (within the instruction) and first suffix position of a block, from its index:
    // block blk covers rows [32*blk, 32*blk+31] of candidate 32*blk / (S*G).
    // A block whose first row is already past its candidate's length holds nothing but padding.
    auto block_cand = [&](int blk) { return WHOLE ? (int)fdiv(fdiv(blk * kBlockRows, a.div_g), a.div_s) : (int)fdiv(blk, div_nb); };
    // (not WHOLE) first row of the block within its candidate, rows that exist from there on
    auto block_row = [&](int blk) { return (blk - block_cand(blk) * nb) * kBlockRows; };
    auto block_rows = [&](int blk) { return WHOLE ? kBlockRows : rows_c - block_row(blk); };
    auto block_i_lo = [&](int blk) {
        return WHOLE ? (int)fdiv(blk * kBlockRows, a.div_g) - block_cand(blk) * a.S : (int)fdiv(block_row(blk), a.div_g);
    };
    auto decode = [&](int blk) __attribute__((always_inline)) {
        if constexpr (WHOLE)
            return decode_block(a, X, blk, X.head, X.cand0);
        const int r = block_row(blk) + X.c32;
        return decode_candidate_row(a, X.cand0 + __builtin_amdgcn_readfirstlane(block_cand(blk)), r < rows_c ? r : rows_c - 1, X.head);
    };
    // Advance to the next block of this wavefront that has a valid row; blocks of pure padding
    // on the way are stored as zeros here and now.
    // Every wavefront takes one contiguous range of blocks, so that a candidate's suffix K/V, which
    // all of its blocks read, is fetched by one compute unit.  The workgroup's share of the virtual
    // head's blocks is cut into four parts, one per SIMD.  The two wavefronts of a SIMD (slots w and
    // w + 4) are not served alike: the one launched first wins the arbitration for the matrix cores
    // and gets through a block about a fifth faster, so it takes 7/12 of the SIMD's part and the
    // other one the rest; with equal shares the second one runs on alone for the last sixth of the
    // launch (measured: 14:10 beats 12:12 by 2-3 %, 13:11 and 15:9 lie between).
    const int wslot = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slice = blockIdx.x / vh_slots;
    const int wg_lo = (int)((long long)nblocks * slice / per_vh), wg_hi = (int)((long long)nblocks * (slice + 1) / per_vh);
    const int simd = wslot & 3;
    const int part_lo = wg_lo + (wg_hi - wg_lo) * simd / 4, part_hi = wg_lo + (wg_hi - wg_lo) * (simd + 1) / 4;
    const int split = part_lo + ((part_hi - part_lo) * 7 + 6) / 12;
    const int blk_lo = wslot < 4 ? part_lo : split, blk_hi = wslot < 4 ? split : part_hi;
    auto skip_padding = [&](int blk) __attribute__((always_inline)) {
        while (blk < blk_hi && block_i_lo(blk) >= len_uniform(a, X.cand0 + block_cand(blk))) {
            store_zero_block_rows(a, X, decode(blk), block_rows(blk));
            ++blk;
        }
        return blk;
    };

    for (int vh = blockIdx.x % vh_slots; vh < VH; vh += vh_slots) {
    set_vhead(a, X, vh);
    const int T = (X.P + kTileKeys - 1) / kTileKeys;

    // first block of this wavefront: request its row decode and Q before the prefix copy
    const int first_blk = blk_lo;
    bool any_bad = false;
    const bool is_short = !WHOLE && T < 3; // this instruction's prefix is too short for the pipeline: see below
    int blk = is_short ? blk_hi : skip_padding(first_blk);
    BlockRows nxt;
    uintx4 q[8]; // this block's Q fragments until their last use, then the next block's
    if (!is_short) {
        nxt = decode(blk < blk_hi ? blk : nblocks - 1);
        load_q_block(a, X, nxt, q);
    }

    __syncthreads(); // every wavefront is done with the images of the virtual head before
    stage_prefix(a, X, T, smem, smem + max_tiles * kTileBytes, tid);
    __syncthreads();

    if constexpr (WHOLE) {
        if (T < 3) { // this instruction's prefix is too short for the pipeline: general path
            for (int b2 = first_blk; b2 < blk_hi; ++b2)
                general_block(a, X, T, b2);
            continue;
        }
    }

    while (blk < blk_hi) {
        const BlockRows row = nxt;
        // the block's suffix step: keys 0..skmax of its candidate
        const int rows = block_rows(blk);
        const int i_hi = WHOLE ? (int)fdiv(blk * kBlockRows + kBlockRows - 1, a.div_g) - (row.b - X.cand0) * a.S
                               : (int)fdiv(rows > kBlockRows ? block_row(blk) + kBlockRows - 1 : rows_c - 1, a.div_g);
        const int skmax = i_hi < row.len - 1 ? i_hi : row.len - 1;
        // Loads are retired in issue order, so what is needed last is requested first.
        uintx4 skf[8], svf[2][4];
        load_suffix_k_block(a, X, row.b, 0, skmax, skf);

        // ---- first prefix tile: scores, reference maximum ----
        floatx16 sA, sB; // raw scores of the current and of the next tile, roles alternating
#pragma unroll
        for (int e = 0; e < 16; ++e)
            sA[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*(lds_u128 *)(X.k_lane + ks * 1024)), as_bf16x8(q[ks]),
                                                         sA, 0, 0, 0);
        Pre pre;
#pragma unroll
        for (int i = 0; i < kDist; ++i)
            pre.k[i] = *(lds_u128 *)(kimg(1) + i * 1024);
        float m = sA[0];
#pragma unroll
        for (int e = 1; e < 16; ++e)
            m = fmaxf(m, sA[e]);
        m = fmaxf(m, __shfl_xor(m, 32, 64)) * X.c; // the other half-wave holds the other 16 keys
        float l = 0.f;
        floatx16 o[4];
        uintx4 pA[2], pB[2]; // packed weights of the current and of the previous tile, roles alternating

        // ---- pipeline over the prefix tiles: step t = scores of tile t+1, weights of tile t,
        //      value product of tile t-1 ----
        pipe_tile<true, false, false, false, false, true, true>(kimg(1), skf, vimg(0), kimg(2), vimg(0), pre, q, sA, sB,
                                                                X.c, m, 0, l, pA, pA, o);
        pipe_tile<true, false, true, true, false, true, true>(kimg(2), skf, vimg(0), kimg(3 < T ? 3 : T - 1), vimg(1), pre,
                                                              q, sB, sA, X.c, m, 0, l, pA, pB, o);
        int t = 2;
        for (; t + 1 <= T - 2; t += 2) {
            pipe_tile<true, false, true, false, false, true, true>(kimg(t + 1), skf, vimg(t - 1), kimg(t + 2), vimg(t), pre,
                                                                   q, sA, sB, X.c, m, 0, l, pB, pA, o);
            pipe_tile<true, false, true, false, false, true, true>(kimg(t + 2), skf, vimg(t), kimg(t + 3 < T ? t + 3 : T - 1),
                                                                   vimg(t + 1), pre, q, sB, sA, X.c, m, 0, l, pA, pB, o);
        }
        if (t <= T - 2) { // one step left over: do it and put scores and weights back in their places
            pipe_tile<true, false, true, false, false, true, true>(kimg(t + 1), skf, vimg(t - 1), kimg(T - 1), vimg(t), pre,
                                                                   q, sA, sB, X.c, m, 0, l, pB, pA, o);
            sA = sB;
            pB[0] = pA[0];
            pB[1] = pA[1];
        }
        if (X.P & (kTileKeys - 1)) { // ragged last prefix tile: keys past the prefix are not visible
            const int nv = X.P - (T - 1) * kTileKeys - 4 * X.h;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if (8 * (e >> 2) + (e & 3) >= nv)
                    sA[e] = -INFINITY;
        }
        load_suffix_v_block(a, X, row.b, 0, skmax, svf); // one step ahead of its use
        // ---- last prefix tile: the "next scores" are the suffix scores, from the K registers ----
        pipe_tile<true, true, true, false, false, false, true>(kimg(0), skf, vimg(T - 2), kimg(0), vimg(T - 1), pre, q, sA,
                                                               sB, X.c, m, 0, l, pB, pA, o);

        // Q has been used for the last time: the next block's row decode and Q take its place.
        // (Requested unconditionally, for a clamped block index past the end: a load under a
        // branch would have to be waited for and copied at the join.)
        blk = skip_padding(blk + 1);
        nxt = decode(blk < blk_hi ? blk : nblocks - 1);
        load_q_block(a, X, nxt, q);

        // ---- suffix step: causal mask and weights under the value product of the last prefix
        //      tile; then the suffix value product through the scratch tile ----
        // the row sees keys 0..ri; element e holds key 8*(e/4) + e%4 + 4*h
        pipe_tile<false, false, true, false, true, false, false>(kimg(0), skf, vimg(T - 1), kimg(0), vimg(0), pre, q, sB, sB,
                                                                 X.c, m, (int)row.ri - 4 * X.h, l, pA, pB, o);
        pv_from_scratch(X, svf[0], as_bf16x8(pB[0]), o);
        pv_from_scratch(X, svf[1], as_bf16x8(pB[1]), o);

        any_bad |= __builtin_amdgcn_ballot_w64(row.ri < row.len && !(l < kBig)) != 0;
        store_block_rows(a, X, row, m, l, o, rows);
    }

    // Rare: some row met scores far above its first tile's maximum.  Whatever this wavefront
    // stored is replaced by the general path's result, its blocks' candidates taken as problems of one candidate.
    // is_short: the general path gains nothing by that and takes the stacked rows' blocks (multi-instruction, 32/8
    // heads, P 96 with prefixes of 60 rows: 400 candidates of 29 positions: 47 us in the general kernel, 57 with own
    // blocks, 48 us so; 24 of 27, 32/32: 10.7, 12.0, 11.5; 23 of 31: 8.4, 11.1, 8.5).
    if constexpr (WHOLE) {
        if (any_bad)
            for (int b2 = first_blk; b2 < blk_hi; ++b2)
                general_block(a, X, T, b2);
    } else if (any_bad || is_short) {
        const int nstacked = (X.Mtot + kBlockRows - 1) / kBlockRows;
        const int share = (int)((unsigned)(nstacked + per_vh - 1) / (unsigned)per_vh); // of a workgroup
        const int end = (slice + 1) * share, hi = !is_short ? blk_hi : end < nstacked ? end : nstacked;
        for (int b2 = is_short ? slice * share + wslot : first_blk; b2 < hi; b2 += is_short ? kNW : 1) {
            Ctx Y = X;
            const int cand = is_short ? 0 : block_cand(b2);
            Y.cand0 = X.cand0 + cand;
            Y.Mtot = is_short ? X.Mtot : rows_c;
            general_block(a, Y, T, b2 - cand * nb);
        }
    }
    } // virtual heads
}

// ------------------------------------------------------------------------------------------
// Pipelined path over packed rows (see pskv_packed.hpp).  Preconditions (checked by the launcher): suffix lengths; S <= 32; a window
// of at most 32 * STEPS positions; a prefix, one head's of less than 2^31 bytes.
//
// Bound by the instructions of a block, as the kernel above, and by memory where the prefix is short; what it gains is blocks: 20480
// instead of 23700 for 1024 candidates of 16..24 of 24 positions, 32/8 heads, P 256 (127.5 -> 118 us; the same with eight instructions 117 -> 110).
// For the same blocks it takes 2 % more vector instructions than that one (512 x 32, P 128: 11.48 million for 11.23; places of rows and keys, masks with two ends).
// Three things cost more than they look: a spilled register's reload in the block loop waits for every request in flight (six of them took back all of the
// gain), a store under a branch makes the wait for the next block's Q one for the stores, and scalars that are kept over everything end up in
// lanes of vector registers (12.87 million vector instructions then).
// Small calls take a workgroup per block while there are compute units: a wavefront alone on its SIMD gets through a block in
// little more than half the time (32 candidates of 20 positions, 32/8 heads, P 128: 11.2 us with eight blocks to a workgroup, 8.5 so; 8.1 by now, 12.4 in the kernels before).
// ------------------------------------------------------------------------------------------
struct PackedLaunch {
    Args a;
    PackedArgs pa;
    int per_vh, vh_slots, max_tiles;
};

// TILES: 1 or 2, the prefix has so many tiles; 3: three and more.  (An instruction whose own prefix has fewer goes the general way.)

template <int STEPS, int TILES>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void resident_packed_kernel(PackedLaunch launch)
{
    extern __shared__ __align__(16) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    // The arguments and all that is made of them are taken anew for every virtual head, and for the general path once more: kept over the
    // loops, 104 to 149 of them were spilled to lanes of vector registers, whose every use is a v_readlane (now 16 to 22, and 236 vector registers for 255;
    // us, before and so: 1024 x 24, 32/8 heads, P 256: 138.2, 137.6; 512 x 20, 32/32, P 128: 74.5, 72.7; 512 x 16..32: 97.8, 94.6).
    auto context = [&](const PackedLaunch &g, int vh) __attribute__((always_inline)) {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        Ctx Y = make_ctx(g.a, smem, g.max_tiles, t);
        set_vhead(g.a, Y, vh);
        return Y;
    };

    const int VH = launch.a.Np * launch.a.Hkv, slots = launch.vh_slots;
    for (int vh = __builtin_amdgcn_readfirstlane(blockIdx.x % slots); vh < VH; vh += slots) {
        const PackedLaunch &launch = first_parameter<PackedLaunch>();
        const Args &a = launch.a;
        const PackedArgs &pa = launch.pa;
        const int per_vh = launch.per_vh, max_tiles = launch.max_tiles;
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        Ctx X = make_ctx(a, smem, max_tiles, tid);
        set_vhead(a, X, vh);
        auto kimg = [&](int t) { return X.k_lane + t * kTileBytes; };
        auto vimg = [&](int t) { return X.v_lane + t * kTileBytes; };
        const int wslot = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int slice = __builtin_amdgcn_readfirstlane(blockIdx.x / launch.vh_slots);
        const int per_chunk = (a.C + kLenChunks - 1) / kLenChunks, waves = per_vh * kNW, me = slice * kNW + wslot;
        lds_int *const lens = (lds_int *)(smem + 2 * max_tiles * kTileBytes); // (in the scratch)
        const int tiles = (X.P + kTileKeys - 1) / kTileKeys;
        const bool fits = TILES == 3 ? tiles >= 3 : tiles == TILES;
        const int T = TILES == 3 ? tiles : TILES; // (of a prefix that fits)
        __syncthreads(); // every wavefront is done with the images and the scratch of the virtual head before

        PackedList list;
        int blk = 0, blk_lo = 0, blk_hi = 0, step = 1; // this wavefront's blocks: from blk_lo, every step-th
        Walk w, begin;
        PackedBlock<STEPS> nxt = {0, 1, X.cand0, 0, 1, 0u, 0u, 0u, 1u, false};
        unsigned q_off = (unsigned)(X.head * a.G) * pa.q_sh;
        uintx4 q[8]; // this block's Q fragments until their last use, then the next block's
        bool any_bad = false;
        // A block's place in an even list.
        auto place = [&](int n) __attribute__((always_inline)) {
            Walk y = walk_even(a, pa.div_run, list.align, n * kBlockRows);
            y.b += X.cand0;
            y.len = list.full ? a.S : packed_len(a, y.b);
            return y;
        };
        // Moves on to the next block whose candidates lie close enough together; w and nxt stay where they are past the last one.
        auto advance = [&](int n) __attribute__((always_inline)) {
            for (; n < blk_hi; n += step) {
                if (step > 1)
                    w = place(n);
                PackedRow row;
                nxt = packed_block<STEPS>(a, pa, X, w, n * kBlockRows, list, q_off, row);
                if (!nxt.wide)
                    break;
                any_bad = true;
            }
            return n;
        };
        // Four wavefronts fetch the lengths and add them up while the other four request the prefix straight into LDS (rows past it
        // take its last row's place).
        int fresh = tid; // (what is worked out from it is not kept over the block loop)
        asm volatile("" : "+v"(fresh));
        if (wslot < kLenWaves) {
            ChunkRows mine = {0, 0};
            for (int k0 = 0; k0 < per_chunk; k0 += kLenRound) {
                int len[kLenRound];
                const int n = per_chunk - k0 < kLenRound ? per_chunk - k0 : kLenRound;
                load_lengths(a, X.cand0, per_chunk, k0, n, fresh, len);
                count_lengths(a, per_chunk, k0, n, len, lens, fresh, mine);
            }
            add_up(mine, lens, fresh);
        } else {
            const TileSlot ts = make_tile_slot(fresh - kLenWaves * 64);
            const unsigned row = (unsigned)a.kp_sp * 2u;
            for (int t = 0; t < tiles; ++t) {
                const int left = X.P - t * kTileKeys - 1; // the last row's place in the tile
                lds_u8 *const at = smem + t * kTileBytes + (wslot - kLenWaves) * 1024;
                const unsigned char *const k0 = reinterpret_cast<const unsigned char *>(X.kpg) + (unsigned)t * kTileKeys * row;
                const unsigned char *const v0 = reinterpret_cast<const unsigned char *>(X.vpg) + (unsigned)t * kTileKeys * row;
                const unsigned ko = (unsigned)(ts.k_row < left ? ts.k_row : left) * row + ts.k_chunk * 16u, vo = (unsigned)(ts.v_row < left ? ts.v_row : left) * row + ts.v_chunk * 16u;
                request_to_lds(k0, ko, at); // (half of the image per request: columns 0..63, then 64..127)
                request_to_lds(k0 + 128, ko, at + kTileBytes / 2);
                request_to_lds(v0, vo, at + max_tiles * kTileBytes);
                request_to_lds(v0 + 128, vo, at + max_tiles * kTileBytes + kTileBytes / 2);
            }
        }
        __syncthreads();
        list = choose_list<STEPS>(a, pa, tiles, waves, per_chunk, lens);
        const int nblocks = (list.total + kBlockRows - 1) / kBlockRows;
        {
            // Contiguous ranges, a quarter of the workgroup's per SIMD, 7/12 of that for the first of its two as in the kernel above, or half where
            // rounding makes that 5 of 8 or 4 of 6 and grouped heads share a candidate's keys (us, 7/12 and half, nothing padded, P 128, 32/8: 256 x 32: 46.9,
            // 42.9; 256 x 24: 37.9, 35.5; 512 x 20: 51.2, 49.5; 32/32: 256 x 24: 48.3, 50.8; 1500 x 24: 254, 263).
            const int each = (int)fdiv(nblocks, pa.div_n), over = nblocks - each * per_vh;
            const int wg_lo = slice * each + (slice < over ? slice : over), wg_n = each + (slice < over ? 1 : 0), simd = wslot & 3;
            const int part_lo = wg_lo + (wg_n * simd >> 2), part_hi = wg_lo + (wg_n * (simd + 1) >> 2), part = part_hi - part_lo;
            const int split = part_lo + (a.G > 1 && part <= 16 ? (part + 1) >> 1 : (part * 7 + 6) / 12);
            blk_lo = wslot < 4 ? part_lo : split, blk_hi = wslot < 4 ? split : part_hi;
            // In turn, neighbouring blocks to neighbouring wavefronts, where places are a division away and bytes bound the call: one block per
            // candidate and key head, or full windows, or a short prefix (us, ranges and in turn: 32/32: 512 x 20, P 128: 72.8, 69.7; 1500 x 24, P 32: 249, 239; 1500 x
            // 32, P 32: 326, 311; 1500 x 22..32: 291, 277; 32/8: 1500 x 28, P 32: 179, 166; 1500 x 24, P 200, not so: 181, 185).
            if (list.even && list.align > 1 && (a.G == 1 || a.S == kTileKeys || TILES < 3)) {
                step = waves;
                blk_lo = me;
                blk_hi = nblocks;
            }
            if (blk_lo < blk_hi)
                begin = w = list.even ? place(blk_lo) : find_row(a, list, X.cand0, blk_lo * kBlockRows, fresh & 63);
            blk = !fits ? blk_hi : advance(blk_lo);
            load_q_packed(a, pa, fresh_lane(X), nxt.b, q_off, q);
        }
        asm volatile("" ::: "memory"); // (Q's eight requests stand before this)
        if (wslot >= kLenWaves) {
            PSKV_WAIT_VM(8);
            if (tiles > 0) { // zeros where the last tile has no row
                const TileSlot ts = make_tile_slot(fresh - kLenWaves * 64);
                const int left = X.P - (tiles - 1) * kTileKeys - 1;
                lds_u8 *const at = smem + (tiles - 1) * kTileBytes + (fresh - kLenWaves * 64) * 16;
                if (ts.k_row > left) {
                    *(lds_u128 *)at = uintx4{0, 0, 0, 0};
                    *(lds_u128 *)(at + kTileBytes / 2) = uintx4{0, 0, 0, 0};
                }
                if (ts.v_row > left) {
                    *(lds_u128 *)(at + max_tiles * kTileBytes) = uintx4{0, 0, 0, 0};
                    *(lds_u128 *)(at + max_tiles * kTileBytes + kTileBytes / 2) = uintx4{0, 0, 0, 0};
                }
            }
        }
        __syncthreads();

        // Padding: the instruction's candidates are dealt out over the wavefronts, and their rows past their lengths stored a
        // few candidates per block.
        int pad = list.full ? a.C : me;
        int shares = (int)fdiv(a.C + waves - 1, pa.div_w);
        asm volatile("" : "+s"(shares));
        const int pads = waves * __builtin_amdgcn_readfirstlane((int)((float)(shares * step) * __builtin_amdgcn_rcpf((float)(blk_hi > blk ? blk_hi - blk : 1))) + 1);

        // The second wavefront of every SIMD begins half a block (some (T + 3) * 0.6 us) later: begun together, the two ask for rows and for the matrix cores at
        // the same times, and in calls of a few blocks they do not drift apart.  Longer calls do by themselves, prefixes of seven tiles and more hide it, and with
        // one block the wait would only be added.  us, together and so, on a card where this shows most (they differ), P 128: 32/32: 512 x 20: 78.0, 74.0; 256 x 14..20:
        // 43.9, 37.8; 512 x 24: 95.1, 87.5; 32/8: 256 x 32: 46.4, 42.4; 512 x 8: 27.0, 23.8; beyond: 1500 x 32: 206, 211; P 256: 512 x 32: 94.7, 97.1.
        if (TILES == 3 && fits && T <= 6 && wslot >= kNW / 2 && nblocks >= 2 * waves && nblocks <= 8 * waves)
            for (int i = 0; i < T + 3; ++i)
                __builtin_amdgcn_s_sleep(11);

        while (blk < blk_hi) {
            const PackedBlock<STEPS> x = nxt;
            // Loads are retired in issue order, so what is needed last is requested first.
            uintx4 skf[8], svf[2][4];
            load_window_k(pa, X, x, 0, skf);

            // ---- first prefix tile: scores, reference maximum ----
            floatx16 sA, sB; // raw scores of the current and of the next tile, roles alternating
#pragma unroll
            for (int e = 0; e < 16; ++e)
                sA[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
                sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*(lds_u128 *)(X.k_lane + ks * 1024)), as_bf16x8(q[ks]),
                                                             sA, 0, 0, 0);
            auto hide_past_prefix = [&]() __attribute__((always_inline)) { // ragged last prefix tile: keys past the prefix are not visible
                if (X.P & (kTileKeys - 1)) {
                    int bits = (1 << (X.P - (T - 1) * kTileKeys)) - 1;
                    bits >>= 4 * fresh_lane(X).h; // element e holds key 8*(e/4) + e%4 + 4*h of the tile
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        sA[e] = hide_unless_bit(sA[e], bits, 8 * (e >> 2) + (e & 3));
                }
            };
            if (TILES == 1)
                hide_past_prefix(); // (before the maximum)
            Pre pre;
            if constexpr (TILES > 1) {
#pragma unroll
                for (int i = 0; i < kDist; ++i)
                    pre.k[i] = *(lds_u128 *)(kimg(1) + i * 1024);
            }
            float m = sA[0];
#pragma unroll
            for (int e = 1; e < 16; ++e)
                m = fmaxf(m, sA[e]);
            m = max_of_halves(m) * X.c; // (the other half-wave holds the other 16 keys)
            // (Stores whose number the compiler does not know stand where the next wait for a load is far: after Q's, before K's.)
            for (const int to = pad + pads < a.C ? pad + pads : a.C; pad < to; pad += waves)
                store_padding(a, fresh_lane(X), X.cand0 + pad, packed_len(a, X.cand0 + pad), list.align, a.out, pa.o_sb, pa.o_ss, pa.o_sh, a.lse);
            float l = 0.f;
            floatx16 o[4];
            uintx4 pA[2], pB[2]; // packed weights of the current and of the previous tile, roles alternating

            // ---- pipeline over the prefix tiles: step t = scores of tile t+1, weights of tile t,
            //      value product of tile t-1 ----
            if constexpr (TILES == 3) {
                pipe_tile<true, false, false, false, 0, true, true>(kimg(1), skf, vimg(0), kimg(2), vimg(0), pre, q, sA, sB,
                                                                    X.c, m, 0, l, pA, pA, o);
                pipe_tile<true, false, true, true, 0, true, true>(kimg(2), skf, vimg(0), added_here(X.k_lane, (3 < T ? 3 : T - 1) * kTileBytes), vimg(1), pre,
                                                                  q, sB, sA, X.c, m, 0, l, pA, pB, o);
                int t = 2;
                for (; t + 1 <= T - 2; t += 2) {
                    pipe_tile<true, false, true, false, 0, true, true>(kimg(t + 1), skf, vimg(t - 1), kimg(t + 2), vimg(t), pre,
                                                                       q, sA, sB, X.c, m, 0, l, pB, pA, o);
                    pipe_tile<true, false, true, false, 0, true, true>(kimg(t + 2), skf, vimg(t), kimg(t + 3 < T ? t + 3 : T - 1),
                                                                       vimg(t + 1), pre, q, sB, sA, X.c, m, 0, l, pA, pB, o);
                }
                if (t <= T - 2) { // one step left over: do it and put scores and weights back in their places
                    pipe_tile<true, false, true, false, 0, true, true>(kimg(t + 1), skf, vimg(t - 1), kimg(T - 1), vimg(t), pre,
                                                                       q, sA, sB, X.c, m, 0, l, pB, pA, o);
                    sA = sB;
                    pB[0] = pA[0];
                    pB[1] = pA[1];
                }
            } else if constexpr (TILES == 2) {
                pipe_tile<true, false, false, false, 0, false, true>(kimg(1), skf, vimg(0), kimg(1), vimg(0), pre, q, sA, sB,
                                                                     X.c, m, 0, l, pA, pB, o);
                sA = sB;
            }
            if (TILES > 1)
                hide_past_prefix();
            load_window_v(pa, X, x, 0, svf); // one step ahead of its use
            lds_u8 *const v_last = added_here(X.v_lane, (T - 1) * kTileBytes);
            // ---- last prefix tile: the "next scores" are the window's first ones, from the K registers ----
            pipe_tile<true, true, (TILES > 1), (TILES == 2), 0, false, true>(kimg(0), skf, TILES == 3 ? added_here(X.v_lane, (T - 2) * kTileBytes) : X.v_lane, kimg(0),
                                                                             v_last, pre, q, sA, sB, X.c, m, 0, l, pB, pA, o);

            // Unless the window goes on, Q has been used for the last time: the next block's rows and Q take its place.
            // (Requested unconditionally, past the end for the last block once more.)
            const bool more = STEPS > 1 && x.width > kTileKeys;
            if (!more) {
                blk = advance(blk + step);
                load_q_packed(a, pa, X, nxt.b, q_off, q);
            }

            // ---- first window step: mask and weights under the value product of the last prefix
            //      tile; then its own value product through the scratch tile ----
            pipe_tile<false, false, true, (TILES == 1), 2, false, false>(kimg(0), skf, v_last, kimg(0), vimg(0), pre, q, sB, sB,
                                                                  X.c, m, sees_bits(x, 0, X.h), l, pA, pB, o);
            const Ctx Y = X;
            if (more)
                load_window_k(pa, Y, x, kTileKeys, skf);
            pv_from_scratch(Y, svf[0], as_bf16x8(pB[0]), o);
            pv_from_scratch(Y, svf[1], as_bf16x8(pB[1]), o);
            if (more) {
                load_window_v(pa, X, x, kTileKeys, svf);
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    sB[e] = 0.f;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks)
                    sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(skf[ks]), as_bf16x8(q[ks]), sB, 0, 0, 0);
                blk = advance(blk + step);
                load_q_packed(a, pa, X, nxt.b, q_off, q);
                window_step_fixed(Y, sees_bits(x, kTileKeys, Y.h), sB, m, l, svf, o);
            }

            any_bad |= __builtin_amdgcn_ballot_w64(!(l < kBig)) != 0;
            store_packed(a, pa, STEPS == 1 || TILES == 1 ? X : fresh_lane(X), x, list.align, m, l, o);
        }
        for (; pad < a.C; pad += waves)
            store_padding(a, fresh_lane(X), X.cand0 + pad, packed_len(a, X.cand0 + pad), list.align, a.out, pa.o_sb, pa.o_ss, pa.o_sh, a.lse);

        // Rare: some row met scores far above its first tile's maximum, or a block's candidates lie far apart: whatever this
        // wavefront stored is replaced by the general path's result.  The same for an instruction whose prefix is too short for
        // the pipeline.
        if (any_bad || !fits) {
            const PackedLaunch &again = first_parameter<PackedLaunch>();
            const Ctx Y = context(again, vh);
            w = begin;
            for (int b2 = blk_lo; b2 < blk_hi; b2 += step) {
                GeneralBlock<2> g;
                packed_general_begin(again.a, again.pa, Y, w, b2 * kBlockRows, list, g);
                for (int kt = 0; kt < tiles; ++kt)
                    prefix_tile_classic(Y, Y.k_lane + kt * kTileBytes, Y.v_lane + kt * kTileBytes, Y.P - kt * kTileKeys, g.q, g.st);
                packed_general_end(again.a, Y, g);
            }
        }
    } // virtual heads
}

} // namespace

bool resident_supported(const Args &a)
{
    return a.D == kD && a.P <= kMaxTiles * kTileKeys;
}

hipError_t launch_resident(const Args &a, hipStream_t stream)
{
    static DeviceSlots cu_by_device;
    hipError_t e;
    const int num_cu = device_setup_once(cu_by_device, e, [] {
        const int max_lds = 2 * kMaxTiles * kTileBytes + kNW * kScrBytes;
        hipError_t s = hipFuncSetAttribute(reinterpret_cast<const void *>(resident_general_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
        for (auto kernel : {resident_pipelined_kernel<true>, resident_pipelined_kernel<false>})
            if (s == hipSuccess)
                s = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
        for (auto kernel : {resident_packed_kernel<2, 1>, resident_packed_kernel<1, 1>, resident_packed_kernel<2, 2>, resident_packed_kernel<1, 2>,
                            resident_packed_kernel<2, 3>, resident_packed_kernel<1, 3>})
            if (s == hipSuccess)
                s = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
        return s;
    });
    if (num_cu == 0)
        return e;
    const int max_tiles = (a.P + kTileKeys - 1) / kTileKeys;
    const long long rows = (long long)a.C * a.S * a.G; // stacked rows of one virtual head
    // Candidates whose rows fill no whole number of blocks: blocks of their own and the pipelined kernel where
    // those come out full to 13/16, the general kernel on full blocks that span candidates where not.  us, general and
    // pipelined: 2048 candidates x 120 rows (8 KV heads, P 100): 265, 227; 1024 x 133 of 160 (4 heads, P 256): 103, 93;
    // 437 x 27 of 32 (32 heads, P 219): 104, 78 (512 x 28, P 128, whose bytes alone take 92: 98, 104); 1024 x 52 of 64 (8 heads, P 200): 84, 78; below: 1024 x 77 of 96: 64,
    // 66; 512 x 24 of 32: 84, 84; 512 x 20 of 32: 65, 67 (P 256: 77, 84); 512 x 12 of 32: 42, 53.
    // Own blocks are more blocks.  A block's time is taken as its tiles and its own step, times 1.7 in the general
    // kernel, which takes one more own step for every candidate that its blocks straddle; the pipelined one has a
    // beginning of four tiles' time.  191 candidates x 84 rows (4 heads, P 75; a wavefront has 1 block or 2): 11.8, 14.3;
    // 94 x 84 (8 heads, P 81; 1, 2): 11.8, 14.4; 89 x 84 (8 heads, P 171; 1, 2): 15.0, 17.8; 24 x 176 (4 heads, P 99;
    // 1, 1): 11.8, 12.6; 148 x 203 (4 heads, P 141; 2, 3): 23.2, 24.0; and 10 x 27 (32 heads, P 151; 1, 1): 13.9,
    // 12.1; 274 x 108 (8 heads, P 153; 4, 5): 44.8, 39.1; 213 x 203 (4 heads, P 142; 3, 3): 30.4, 28.2.
    const long long rows_c = (long long)a.S * a.G, nb = (rows_c + kBlockRows - 1) / kBlockRows; // rows and own blocks of a candidate
    const long long stacked = (rows + kBlockRows - 1) / kBlockRows, own = a.C * nb;
    const bool whole = rows_c % kBlockRows == 0;
    bool pipelined = a.S <= kTileKeys && max_tiles >= 3 && block_offsets_fit(a) && rows_c * 16 >= nb * kBlockRows * 13 &&
                     own <= 0x7fffffffLL / kBlockRows;
    if (pipelined && !whole) {
        const double straddled = rows_c < kBlockRows ? 1. : (double)kBlockRows / rows_c;
        const long long each_own = resident_split(a, own, kNW, num_cu).each, each_stacked = resident_split(a, stacked, kNW, num_cu).each;
        pipelined = each_own * (max_tiles + 1) + 4 <= 1.7 * each_stacked * (max_tiles + 1 + straddled);
    }
    // Rows packed by their lengths, where there are lengths: us, in the kernels above and so: 32/8 heads: 1500 x 20, P 200: 179, 152; 1500 x 8..20: 146, 116; 500 x 28,
    // P 250: 93, 85; 700 x 28, P 128: 94.9, 93.7; 32/32: 1500 x 14, P 200: 187, 158; 512 x 20, P 128: 76.5, 73.9 (its bytes alone take 66); 700 x 22..32, P 128: 147,
    // 143; 28/4: 200 x 28, P 100: 32.3, 27.9; 8 x 12..24, 32/8, P 100: 11.5, 7.2; prefixes of one tile or two: 300 x 20, P 40, 32/8: 33.3, 30.4; 600 x 10..20, P 64:
    // 54.6, 48.0.  Nothing to pack: 500 x 32, 32/8, P 250: 93.3, 93.9; 1500 x 32, P 200: 240, 244; 1500 x 24: 183, 182; 1500 x 32, 32/32, P 32: 313, 310; what is left
    // below is 1500 x 24, 32/32, P 128: 247, 259 (512 x 24: 87.0, 87.5) and 28/4 heads of 32 positions: 256 x 32, P 192: 44.6, 45.7.
    PackedArgs pa;
    const ResidentSplit packed = resident_split(a, own * kNW, kNW, num_cu); // (a workgroup per block while there are compute units)
    if (a.len && max_tiles >= 1 && a.S <= kTileKeys && own <= 0x7fffffffLL / kBlockRows && (long long)a.P * a.kp_sp * 2 < 0x7fffffffLL && packed_args(a, (unsigned)packed.per_vh, kNW, pa)) {
        const bool two = packed_steps(a, 2, pa.dense) > 1;
        auto kernel = max_tiles == 1 ? (two ? resident_packed_kernel<2, 1> : resident_packed_kernel<1, 1>)
                      : max_tiles == 2 ? (two ? resident_packed_kernel<2, 2> : resident_packed_kernel<1, 2>)
                                       : (two ? resident_packed_kernel<2, 3> : resident_packed_kernel<1, 3>);
        return launch_kernel(kernel,
                             dim3((unsigned)(packed.per_vh * packed.vh_slots)), dim3(kNW * 64), (size_t)2 * max_tiles * kTileBytes + kNW * kScrBytes,
                             stream, PackedLaunch{a, pa, (int)packed.per_vh, (int)packed.vh_slots, max_tiles});
    }
    // One workgroup per compute unit.
    const ResidentSplit split = resident_split(a, pipelined ? own : stacked, kNW, num_cu);
    const int per_vh = (int)split.per_vh, vh_slots = (int)split.vh_slots;
    const unsigned grid = (unsigned)(split.per_vh * split.vh_slots);
    const size_t lds = (size_t)2 * max_tiles * kTileBytes + kNW * kScrBytes;
    if (pipelined)
        return launch_kernel(whole ? resident_pipelined_kernel<true> : resident_pipelined_kernel<false>, dim3(grid), dim3(kNW * 64),
                             lds, stream, a, per_vh, vh_slots, max_tiles, (int)nb, make_fastdiv((unsigned)nb));
    else
        return launch_kernel(resident_general_kernel, dim3(grid), dim3(kNW * 64), lds, stream, a, per_vh,
                           vh_slots, max_tiles);
}

} // namespace pskv
