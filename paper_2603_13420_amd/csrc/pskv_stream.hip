// Streamed-prefix MFMA kernels of batched candidate-suffix attention for gfx950
// (bf16 tensors, head dim 128, prefix of any length).
//
// Used when the prefix K/V of one head does not fit in LDS.  The stacked query rows
//     r = (b*S + i)*G + g      (suffix-centric alignment, Sec. 4.3)
// of one KV head are cut into groups of 256; a "pass" is one (KV head, group) pair.  A
// persistent workgroup of 8 wavefronts takes passes in turn; each wavefront owns one 32-row
// block of the group and all eight walk over the prefix together, tile by tile: the 512 threads
// request the coming 32-key tiles of the single shared prefix K/V (Sec. 4.2: one copy for all
// candidates) from L2 straight into a small ring of fragment-major LDS images while the current
// tiles are being used, and meet at one barrier per two tiles.  Every tile is thus
// read once per 256 rows, whatever candidates those rows belong to, and the prefix itself is
// read from HBM about once per XCD: pass ids are laid out so that the workgroups of one XCD
// (workgroup ids go round the XCDs) work on one head at a time, and find it in that XCD's L2.
//
// Five kernels.  The pipelined one (every 32-row block inside one candidate) is the software
// pipeline of the resident-prefix kernel with the tile images taken from the ring, the suffix
// handled after the prefix, and a fixed per-row reference maximum; when a row turns out to
// need rescaling, the workgroup repeats its passes on the general path.  The general one
// (any shape) is the classic online softmax, one tile at a time.  The third (further down) is
// for suffix-side segments of several tiles: its passes are cut out of one candidate, whose own
// suffix K/V then goes through the ring like the prefix.  The fourth is the third with passes of half the size, two at
// a time on a compute unit.  The fifth is the pipelined one with blocks of valid rows only (pskv_packed.hpp).
// Operand layouts and the pieces shared with the resident kernels are in pskv_mfma.hpp.
#include "pskv_packed.hpp"

namespace pskv {
namespace {

constexpr int kRing = 8;                   // tile slots in LDS
constexpr int kSlotBytes = 2 * kTileBytes; // K image, then V image
constexpr int kLdsBytes = kRing * kSlotBytes + kNW * kScrBytes;
constexpr int kPassRows = kNW * kBlockRows;
constexpr int kMinTiles = 3;                // shortest prefix, in tiles, that the pipelined pass takes

typedef __attribute__((address_space(3))) int lds_int;

__device__ inline Ctx make_stream_ctx(const Args &a, lds_u8 *smem, int tid)
{
    Ctx X;
    X.lane = tid & 63;
    X.h = X.lane >> 5;
    X.c32 = X.lane & 31;
    X.Mtot = a.C * a.S * a.G;
    X.c = a.scale * kLog2e;
    X.k_lane = smem + X.lane * 16;             // slot 0; slot s is kSlotBytes*s further
    X.v_lane = smem + kTileBytes + X.lane * 8;
    X.scr = smem + kRing * kSlotBytes + __builtin_amdgcn_readfirstlane(tid >> 6) * kScrBytes;
    X.sv_row_lo = 4 * ((X.c32 >> 4) & 1) + ((X.c32 >> 1) & 3);
    X.sv_chunk_lo = 2 * ((X.c32 >> 3) & 1) + (X.c32 & 1);
    set_vhead(a, X, 0);
    return X;
}

// ------------------------------------------------------------------------------------------
// General pass: classic online softmax, tiles double-buffered in slots 0 and 1.  Every thread
// of the workgroup must call it (barriers inside), whether or not its wavefront has a block.
// cand, rows_c: with rows_c > 0, blk counts within that candidate of the instruction, a problem of its own.
// ------------------------------------------------------------------------------------------
template <int THREADS = 512>
__device__ __attribute__((always_inline)) void general_pass(const Args &a, Ctx &X, lds_u8 *smem, int tid, int vh, int blk,
                                                            bool active, int cand = 0, int rows_c = 0)
{
    set_vhead(a, X, vh);
    if (rows_c > 0) {
        X.cand0 += cand;
        X.Mtot = rows_c;
    }
    const int ntiles = (X.P + kTileKeys - 1) / kTileKeys;
    constexpr int kParts = 512 / THREADS; // chunks of a tile's K, and of its V, per thread
    TileSlot t[kParts];
#pragma unroll
    for (int i = 0; i < kParts; ++i)
        t[i] = make_tile_slot(tid + i * THREADS);
    const int r0 = blk * kBlockRows;
    const Row row = decode_row(a, X, blk);
    const bool rvalid = active && row.rin && (int)row.ri < clamp_len(a, row.rlen);
    const bool work = __builtin_amdgcn_ballot_w64(rvalid) != 0;
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

    if (ntiles > 0) {
        uintx4 kv[kParts], vv[kParts];
        auto load = [&](int kt) {
#pragma unroll
            for (int i = 0; i < kParts; ++i)
                load_tile_chunks(a, X, t[i], kt, kv[i], vv[i]);
        };
        auto write = [&](int kt, lds_u8 *slot) {
#pragma unroll
            for (int i = 0; i < kParts; ++i)
                write_tile_chunks(X, t[i], kt, slot, slot + kTileBytes, tid + i * THREADS, kv[i], vv[i]);
        };
        load(0);
        __syncthreads(); // whatever the ring held has been used by every wavefront
        write(0, smem);
        __syncthreads();
        for (int kt = 0; kt < ntiles; ++kt) {
            load(kt + 1 < ntiles ? kt + 1 : kt);
            if (work)
                prefix_tile_classic(X, X.k_lane + (kt & 1) * kSlotBytes, X.v_lane + (kt & 1) * kSlotBytes,
                                    X.P - kt * kTileKeys, q, st);
            if (kt + 1 < ntiles)
                write(kt + 1, smem + ((kt + 1) & 1) * kSlotBytes);
            __syncthreads();
        }
    }
    if (active) {
        if (work) {
            suffix_classic(a, X, r0, row, q, st);
            store_block(a, X, r0, row, rvalid, st.m, st.l, st.o);
        } else {
            store_zero_block(a, X, r0, row);
        }
    }
}

__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void stream_general_kernel(Args a, int npasses)
{
    extern __shared__ __align__(16) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X = make_stream_ctx(a, smem, tid);
    const int nblocks = (X.Mtot + kBlockRows - 1) / kBlockRows;
    for (int p = blockIdx.x; p < npasses; p += gridDim.x) {
        const Pass ps = make_pass(a, p, npasses, nblocks, wave);
        if (ps.exists)
            general_pass(a, X, smem, tid, ps.vh, ps.blk, ps.active);
    }
}

// ------------------------------------------------------------------------------------------
// Pipelined passes.  Preconditions (checked by the launcher): every 32-row block lies inside one candidate; the padded prefix has at least three tiles; one head's prefix
// spans less than 2^31 bytes, so tile addresses are a scalar base plus a 32-bit lane offset.
// ONE_STEP: S <= 32, the suffix is a single 32-key step.
// WHOLE: S*G is a multiple of 32, the blocks are those of the stacked rows.  Otherwise a candidate has nb
// blocks of its own, the last one being what is left (its rows past the candidate's stand in for the last
// one and are not stored), here and in the candidate passes further down.
//
// Ring protocol.  Step t of a pass (see pipe_tile) reads the K images of tiles t+1 and t+2 and
// the V images of tiles t-1 and t.  Steps are taken two at a time.  Tiles are requested with
// direct-to-LDS loads, tile u into slot u % 8, tiles 0..6 at the start of the pass.  At the top
// of the pair (t, t+1) every thread waits until its requests for the tiles up to t+3 have landed
// (the vector memory counter retires requests in order: all but those of tile t+4 must be
// complete), the workgroup meets at a barrier - after which everybody's parts of those tiles are
// there and nobody reads tiles up to t-2 any more - and tiles t+5 and t+6 are requested into the
// slots of tiles t-3 and t-2.  The pair then reads tiles t-1 .. t+3.
// Rows past the end of a ragged last tile are fetched from the last prefix row instead: their
// scores are masked and their weights are exactly zero, so finite data is all that is needed.
// ------------------------------------------------------------------------------------------
struct Stager {
    const unsigned char *kbase, *vbase; // this head's prefix K and V (wave-uniform)
    unsigned k_off, v_off;              // this thread's chunk within a full tile, bytes
    unsigned k_off_last, v_off_last;    // ... within the last tile (rows clamped into the prefix)
    unsigned tile_stride;               // bytes from one tile to the next
    int last;                           // index of the last tile
};

template <bool WHOLE> __device__ inline BlockRows decode_own(const Args &a, const Ctx &X, int blk, int head, int cand0, int cand, int nb)
{
    if constexpr (WHOLE)
        return decode_block(a, X, blk, head, cand0);
    const int rows_c = a.S * a.G, r = (blk - cand * nb) * kBlockRows + X.c32;
    return decode_candidate_row(a, cand0 + __builtin_amdgcn_readfirstlane(cand), r < rows_c ? r : rows_c - 1, head);
}

template <bool ONE_STEP, bool WHOLE>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void stream_pipelined_kernel(Args a, int npasses, int nb, FastDiv div_nb)
{
    extern __shared__ __align__(16) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X = make_stream_ctx(a, smem, tid);
    const int rows_c = a.S * a.G; // rows of a candidate
    const int nblocks = WHOLE ? (X.Mtot + kBlockRows - 1) / kBlockRows : a.C * nb;
    auto cand_of = [&](int blk) { return WHOLE ? 0 : (int)fdiv(blk, div_nb); }; // (not WHOLE) candidate within the instruction
    auto decode = [&](const Pass &ps) __attribute__((always_inline)) {
        return decode_own<WHOLE>(a, X, ps.blk, ps.head, ps.cand0, cand_of(ps.blk), nb);
    };
    auto kimg = [&](int t) { return X.k_lane + (t & (kRing - 1)) * kSlotBytes; };
    auto vimg = [&](int t) { return X.v_lane + (t & (kRing - 1)) * kSlotBytes; };
    // this thread's two requests for tile kt (kt <= the last tile), straight into slot kt % 8
    auto request = [&](const Stager &g, int kt) {
        const unsigned base = (unsigned)kt * g.tile_stride;
        lds_u8 *slot = smem + (kt & (kRing - 1)) * kSlotBytes + wave * 1024;
        request_to_lds(g.kbase + base, kt == g.last ? g.k_off_last : g.k_off, slot);
        request_to_lds(g.vbase + base, kt == g.last ? g.v_off_last : g.v_off, slot + kTileBytes);
    };

    Stager g;
    const TileSlot ts = make_tile_slot(tid);
    g.k_off = (unsigned)(ts.k_row * a.kp_sp + ts.k_chunk * 8) * 2u;
    g.v_off = (unsigned)(ts.v_row * a.kp_sp + ts.v_chunk * 8) * 2u;
    g.tile_stride = (unsigned)(kTileKeys * a.kp_sp) * 2u;

    bool wg_bad = false;
    int p = blockIdx.x;
    Pass ps = make_pass(a, p, npasses, nblocks, wave);
    BlockRows nxt = decode(ps);
    uintx4 q[8]; // this pass's Q fragments until their last use, then the next pass's
    load_q_block(a, X, nxt, q);

    bool wg_short = false;
    while (p < npasses) {
        set_vhead(a, X, ps.vh);
        const int T = (X.P + kTileKeys - 1) / kTileKeys;
        if (!ps.exists || T < kMinTiles) { // nothing here, or this instruction's prefix is too short for the pipeline:
                                           // left to the general sweep below
            wg_short |= ps.exists;
            p += gridDim.x;
            ps = make_pass(a, p, npasses, nblocks, wave);
            nxt = decode(ps);
            load_q_block(a, X, nxt, q);
            continue;
        }
        {
            const int nlast = X.P - (T - 1) * kTileKeys; // rows of the last tile, 1..32
            const int kr = ts.k_row < nlast ? ts.k_row : nlast - 1, vr = ts.v_row < nlast ? ts.v_row : nlast - 1;
            g.k_off_last = (unsigned)(kr * a.kp_sp + ts.k_chunk * 8) * 2u;
            g.v_off_last = (unsigned)(vr * a.kp_sp + ts.v_chunk * 8) * 2u;
            g.last = T - 1;
            g.kbase = reinterpret_cast<const unsigned char *>(X.kpg);
            g.vbase = reinterpret_cast<const unsigned char *>(X.vpg);
        }
        const int blk = ps.blk, r0 = blk * kBlockRows;
        const bool active = ps.active;
        const BlockRows row = nxt;
        const bool rvalid = active && row.ri < row.len;

        // The ring is free here: the barrier that ended the previous pass was passed only by
        // wavefronts that had finished reading it.  Tiles 0..6 are requested at once; the first
        // steps need tiles 0..3.
#pragma unroll
        for (int u = 0; u < 7; ++u)
            if (u < T)
                request(g, u);
        if (T >= 7)
            PSKV_WAIT_VM(6);
        else
            PSKV_WAIT_VM(0);
        __syncthreads();
        // Top of the pair (t, t+1): tiles up to t+3 have landed for everyone (tile t+4 may still be
        // in flight); nobody reads tiles up to t-2 any more: their slots take tiles t+5 and t+6.
        auto pair_top = [&](int t) {
            if (t + 4 <= T - 1)
                PSKV_WAIT_VM(2);
            else
                PSKV_WAIT_VM(0);
            __syncthreads();
            if (t + 5 <= T - 1)
                request(g, t + 5);
            if (t + 6 <= T - 1)
                request(g, t + 6);
        };

        // the block's suffix: candidate sb, keys 0..skmax
        const int r_own = WHOLE ? 0 : r0 - cand_of(blk) * nb * kBlockRows; // (not WHOLE) first row within the candidate
        const int rows = WHOLE ? kBlockRows : rows_c - r_own;
        const int i_hi = WHOLE ? (int)fdiv(r0 + kBlockRows - 1, a.div_g) - (row.b - X.cand0) * a.S
                               : (int)fdiv(r_own + kBlockRows - 1, a.div_g);
        const int skmax = i_hi < row.len - 1 ? i_hi : row.len - 1;
        const int skld = skmax > 0 ? skmax : 0; // row the suffix loads are clamped to (a candidate may be empty)

        // ---- first prefix tile: scores, reference maximum ----
        floatx16 sA, sB; // raw scores of the current and of the next tile, roles alternating
#pragma unroll
        for (int e = 0; e < 16; ++e)
            sA[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*(lds_u128 *)(kimg(0) + ks * 1024)), as_bf16x8(q[ks]), sA,
                                                         0, 0, 0);
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
        uintx4 skf[8], svf[2][4];

        // ---- pipeline over the prefix tiles: step t = scores of tile t+1, weights of tile t,
        //      value product of tile t-1 ----
        pipe_tile<true, false, false, false, false, true, true>(kimg(1), skf, vimg(0), kimg(2), vimg(0), pre, q, sA, sB,
                                                                X.c, m, 0, l, pA, pA, o);
        pipe_tile<true, false, true, true, false, true, true>(kimg(2), skf, vimg(0), kimg(3), vimg(1), pre, q, sB, sA, X.c,
                                                              m, 0, l, pA, pB, o);
        // one pair of steps
#define PSKV_STEP_PAIR(t)                                                                                              \
    do {                                                                                                               \
        pipe_tile<true, false, true, false, false, true, true>(kimg((t) + 1), skf, vimg((t) - 1), kimg((t) + 2),       \
                                                               vimg(t), pre, q, sA, sB, X.c, m, 0, l, pB, pA, o);      \
        pipe_tile<true, false, true, false, false, true, true>(kimg((t) + 2), skf, vimg(t),                            \
                                                               kimg((t) + 3 < T ? (t) + 3 : T - 1), vimg((t) + 1),     \
                                                               pre, q, sB, sA, X.c, m, 0, l, pA, pB, o);               \
    } while (0)
        int t = 2;
        for (; t + 3 <= T - 2; t += 2) {
            pair_top(t);
            PSKV_STEP_PAIR(t);
        }
        // The last pair requests no further tiles; the suffix K fragments, needed two or three
        // steps from here, are requested once the staging registers are free.
        if (t + 1 <= T - 2) {
            pair_top(t);
            load_suffix_k_block(a, X, row.b, 0, skld, skf);
            PSKV_STEP_PAIR(t);
            t += 2;
        } else {
            load_suffix_k_block(a, X, row.b, 0, skld, skf);
        }
#undef PSKV_STEP_PAIR
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
        load_suffix_v_block(a, X, row.b, 0, skld, svf); // one step ahead of its use
        // ---- last prefix tile: the "next scores" are those of the first suffix step ----
        pipe_tile<true, true, true, false, false, false, true>(kimg(0), skf, vimg(T - 2), kimg(0), vimg(T - 1), pre, q, sA,
                                                               sB, X.c, m, 0, l, pB, pA, o);

        // the next pass of this workgroup (clamped past the end: requested unconditionally)
        p += gridDim.x;
        ps = make_pass(a, p, npasses, nblocks, wave);
        // Without further suffix steps (always so when S <= 32) Q has been used for the last time:
        // the next pass's Q takes its place.
        const bool more = !ONE_STEP && skmax >= kTileKeys;
        if (!more) {
            nxt = decode(ps);
            load_q_block(a, X, nxt, q);
        }

        // ---- first suffix step: causal mask and weights under the value product of the last
        //      prefix tile; then its own value product through the scratch tile ----
        pipe_tile<false, false, true, false, true, false, false>(kimg(0), skf, vimg(T - 1), kimg(0), vimg(0), pre, q, sB, sB,
                                                                 X.c, m, row.ri - 4 * X.h, l, pA, pB, o);
        pv_from_scratch(X, svf[0], as_bf16x8(pB[0]), o);
        pv_from_scratch(X, svf[1], as_bf16x8(pB[1]), o);
        if (more) {
            // The second suffix step's K and V and, in the same round trip to memory, the next
            // pass's Q (into registers of its own: this pass's Q is still needed for the scores).
            uintx4 qn[8];
            load_suffix_k_block(a, X, row.b, kTileKeys, skmax, skf);
            load_suffix_v_block(a, X, row.b, kTileKeys, skmax, svf);
            nxt = decode(ps);
            load_q_block(a, X, nxt, qn);
            for (int k0 = kTileKeys;; k0 += kTileKeys) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    sB[e] = 0.f;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks)
                    sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(skf[ks]), as_bf16x8(q[ks]), sB, 0, 0, 0);
                const bool again = k0 + kTileKeys <= skmax;
                if (again)
                    load_suffix_k_block(a, X, row.b, k0 + kTileKeys, skmax, skf);
                suffix_step_fixed(X, row.ri, k0, sB, m, l, svf, o);
                if (!again)
                    break;
                load_suffix_v_block(a, X, row.b, k0 + kTileKeys, skmax, svf);
            }
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
                q[ks] = qn[ks];
        }

        const bool bad = __builtin_amdgcn_ballot_w64(rvalid && !(l < kBig)) != 0;
        if (active)
            store_block_rows(a, X, row, m, l, o, rows);
        // the wavefront's verdict goes into the first word of its own scratch tile
        if (X.lane == 0)
            *(lds_int *)X.scr = bad ? 1 : 0;
        __syncthreads(); // ends the pass: the ring is free, the verdicts are visible
        wg_bad |= __builtin_amdgcn_ballot_w64(*(lds_int *)(smem + kRing * kSlotBytes + (X.lane & (kNW - 1)) * kScrBytes) !=
                                              0) != 0;
    }

    // Rare: some row met scores far above its first tile's maximum; whatever this workgroup
    // stored is then replaced by the general path's result.  The same sweep serves the passes
    // skipped above.  (Kept out of the main loop so that it costs it no registers.)
    if (wg_bad || wg_short)
        for (int p2 = blockIdx.x; p2 < npasses; p2 += gridDim.x) {
            const Pass ps2 = make_pass(a, p2, npasses, nblocks, wave);
            set_vhead(a, X, ps2.vh);
            if (ps2.exists && (wg_bad || (X.P + kTileKeys - 1) / kTileKeys < kMinTiles))
                general_pass(a, X, smem, tid, ps2.vh, ps2.blk - cand_of(ps2.blk) * nb, ps2.active, cand_of(ps2.blk), WHOLE ? 0 : rows_c);
        }
}

// ------------------------------------------------------------------------------------------
// Pipelined passes over packed rows (pskv_packed.hpp): calls with one prefix and suffix lengths, S <= 64, in place of the
// pipelined kernel above.  A pass is `waves` blocks of one KV head's list (the same list for every head), eight unless
// there are fewer passes than compute units; wavefronts without a block only stage.  Windows of up to STEPS steps.
//
// Bound as the pipelined kernel, tile steps and, at a pass' ends, waits that all of the workgroup shares; what it gains is passes:
// 4096 candidates of 32..64 positions, 40/40 heads, P 512: 246 thousand blocks for 328 thousand, 3742 -> 3254 us, although a block's
// window takes 2.3 steps instead of 1.5.  A pass costs more than there: the search for its first candidate (64 lengths at a time, asked
// for two steps before), the places of rows and keys, and one length per wavefront of a candidate whose padding it stores.
// Tried: the next pass's Q asked for in one place before the window's steps, with this pass's kept or fetched again for the later ones:
// 46 to 69 registers spilled, 0.82 of the pipelined kernel's speed there; asked for after the store it was slower, too.  As it is its
// loads stand under two branches.
// ------------------------------------------------------------------------------------------
struct PackedPass {
    int head, blk; // KV head, this wavefront's block
    bool exists;   // the pass id holds an item (the same for the whole workgroup)
    bool active;   // ... and this wavefront has a block
};

__device__ inline PackedPass packed_pass(const Args &a, int p, int npasses, int nblocks, int waves, int wave)
{
    PackedPass ps;
    const int ngroups = (nblocks + waves - 1) / waves, items = a.Hkv * ngroups;
    const int x = p & 7, y = p >> 3; // (ids as in make_pass)
    const int item = ngroups < kLongHead ? x * ((items + 7) >> 3) + y : ((y / kChunk) * 8 + x) * kChunk + y % kChunk;
    ps.exists = p < npasses && item < items && (ngroups >= kLongHead || y < (items + 7) >> 3);
    const int hpos = ps.exists ? item / ngroups : 0, group = ps.exists ? item - hpos * ngroups : 0;
    const int nfull = a.Hkv >> 3, rem = a.Hkv & 7, cut = rem * (nfull + 1); // (heads in the order 0, 8, ..., 1, 9, ...)
    const int r = hpos < cut ? hpos / (nfull + 1) : rem + (hpos - cut) / (nfull > 0 ? nfull : 1);
    ps.head = (hpos < cut ? hpos - r * (nfull + 1) : (hpos - cut) - (r - rem) * nfull) * 8 + r;
    ps.blk = group * waves + wave;
    ps.active = ps.exists && wave < waves && ps.blk < nblocks;
    return ps;
}

// Where a row of the list is looked for.
struct RowSearch {
    int cand, base; // first candidate, the rows before it
    int len;        // lane j: length of candidate cand + j (0 past the last one)
};

struct StreamPacked {
    Args a;
    PackedArgs pa;
};

template <int STEPS>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void stream_packed_kernel(StreamPacked call)
{
    const Args &a = call.a;
    const PackedArgs &pa = call.pa;
    extern __shared__ __align__(16) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X = make_stream_ctx(a, smem, tid);
    auto kimg = [&](int t) { return X.k_lane + (t & (kRing - 1)) * kSlotBytes; };
    auto vimg = [&](int t) { return X.v_lane + (t & (kRing - 1)) * kSlotBytes; };
    const int T = (a.P + kTileKeys - 1) / kTileKeys;

    // The list of rows, added up in the ring's place; what the passes need of it stays in a register per lane.
    const int per_chunk = (a.C + kLenChunks - 1) / kLenChunks;
    int upto;
    PackedList list;
    {
        lds_int *const lens = (lds_int *)smem;
        if (wave < kLenWaves) {
            ChunkRows mine = {0, 0};
            for (int k0 = 0; k0 < per_chunk; k0 += kLenRound) {
                int len[kLenRound];
                const int n = per_chunk - k0 < kLenRound ? per_chunk - k0 : kLenRound;
                load_lengths(a, 0, per_chunk, k0, n, tid, len);
                count_lengths(a, per_chunk, k0, n, len, lens, tid, mine);
            }
            add_up(mine, lens, tid);
        }
        __syncthreads();
        list = choose_list<STEPS>(a, pa, T, 0, per_chunk, lens);
        upto = rows_upto(list, tid & 63);
        __syncthreads();
    }
    const int nblocks = (list.total + kBlockRows - 1) / kBlockRows;
    int waves = kNW; // blocks of a pass
    while (waves > 1 && (long long)a.Hkv * ((nblocks + waves / 2 - 1) / (waves / 2)) <= gridDim.x)
        waves /= 2;
    const int ngroups = (nblocks + waves - 1) / waves;
    const int npasses = (int)(8 * pass_ids_per_xcd((long long)a.Hkv * ngroups, ngroups));

    // Padding: every pair of a KV head and a candidate belongs to one wavefront, which stores some at the end of each pass.
    const int all_waves = gridDim.x * kNW, pairs = a.Hkv * a.C;
    int pair = list.even ? pairs : blockIdx.x * kNW + wave, pair_head = pair / a.C, pair_cand = pair - pair_head * a.C;
    const int step_head = all_waves / a.C, step_cand = all_waves - step_head * a.C;
    const int shares = (pairs + all_waves - 1) / all_waves, passes = (npasses + (int)gridDim.x - 1) / (int)gridDim.x;
    const int each = __builtin_amdgcn_readfirstlane(shares / (passes > 0 ? passes : 1)) + 1;
    auto pair_len = [&](const Args &a) { return pair < pairs ? packed_len(a, pair_cand) : 0; };
    auto store_pair = [&](const Args &a, const PackedArgs &pa, int len) __attribute__((always_inline)) {
        Ctx Y = fresh_lane(X);
        Y.head = pair_head;
        store_padding(a, Y, pair_cand, len, list.align, a.out, pa.o_sb, pa.o_ss, pa.o_sh, a.lse);
        pair += all_waves;
        pair_head += step_head;
        pair_cand += step_cand;
        if (pair_cand >= a.C) {
            pair_cand -= a.C;
            ++pair_head;
        }
    };

    auto lengths_from = [&](const Args &a, int cand) __attribute__((always_inline)) {
        const int c = cand + fresh_lane(X).lane, len = a.len[c < a.C ? c : a.C - 1];
        return c < a.C ? len : 0;
    };
    auto search_begin = [&](const Args &a, int r0) __attribute__((always_inline)) {
        RowSearch z = {0, 0, 0};
        if (list.even)
            return z;
        const int g = __builtin_popcountll(__builtin_amdgcn_ballot_w64(upto <= r0));
        z.base = g > 0 ? __builtin_amdgcn_readlane(upto, g > 0 ? g - 1 : 0) : 0;
        z.cand = __builtin_amdgcn_readfirstlane(g * kLenPerLane * per_chunk);
        z.len = lengths_from(a, z.cand);
        return z;
    };
    auto search_end = [&](const Args &a, RowSearch &z, int r0) __attribute__((always_inline)) {
        Walk w;
        for (;;) {
            z.len = clamp_len(a, z.len);
            const int sum = wave_scan(packed_run(a, z.len, list.align)), all = __builtin_amdgcn_readlane(sum, 63);
            const int left = a.C - 1 - z.cand < 63 ? a.C - 1 - z.cand : 63; // (the last candidate ends it, whatever the lengths say)
            if (z.base + all > r0 || left < 63) {
                int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(z.base + sum <= r0));
                c = c < left ? c : left;
                w.b = z.cand + c;
                w.first = z.base + (c > 0 ? __builtin_amdgcn_readlane(sum, c > 0 ? c - 1 : 0) : 0);
                w.len = __builtin_amdgcn_readlane(z.len, c);
                return w;
            }
            z.base += all; // (64 at a time: 4096 candidates and more)
            z.cand += 64;
            z.len = lengths_from(a, z.cand);
        }
    };

    auto find = [&](const Args &a, const PackedArgs &pa, RowSearch &z, int r0) __attribute__((always_inline)) {
        if (!list.even)
            return search_end(a, z, r0);
        Walk w = walk_even(a, pa.div_run, list.align, r0);
        w.len = packed_len(a, w.b);
        return w;
    };

    // this thread's two requests for tile kt (kt <= the last tile), straight into slot kt % 8
    const TileSlot ts = make_tile_slot(tid);
    const unsigned row_bytes = (unsigned)a.kp_sp * 2u;
    const unsigned k_off = (unsigned)ts.k_row * row_bytes + ts.k_chunk * 16u, v_off = (unsigned)ts.v_row * row_bytes + ts.v_chunk * 16u;
    const int past = T * kTileKeys - a.P; // rows that the last tile lacks
    auto request = [&](int kt) {
        const unsigned base = (unsigned)kt * kTileKeys * row_bytes;
        lds_u8 *slot = smem + (kt & (kRing - 1)) * kSlotBytes + wave * 1024;
        unsigned ko = k_off, vo = v_off;
        if (kt == T - 1 && past) { // (rows past the prefix: its last one; never visible)
            int t2 = tid;
            asm volatile("" : "+v"(t2));
            const TileSlot t = make_tile_slot(t2);
            const int lastr = kTileKeys - 1 - past;
            ko -= (unsigned)(t.k_row > lastr ? t.k_row - lastr : 0) * row_bytes;
            vo -= (unsigned)(t.v_row > lastr ? t.v_row - lastr : 0) * row_bytes;
        }
        request_to_lds(reinterpret_cast<const unsigned char *>(X.kpg) + base, ko, slot);
        request_to_lds(reinterpret_cast<const unsigned char *>(X.vpg) + base, vo, slot + kTileBytes);
    };
    // The ring protocol is that of the kernel above.
    auto pass_top = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 7; ++u)
            if (u < T)
                request(u);
        if (T >= 7)
            PSKV_WAIT_VM(6);
        else
            PSKV_WAIT_VM(0);
        __syncthreads();
    };
    auto pair_top = [&](int t) __attribute__((always_inline)) {
        if (t + 4 <= T - 1)
            PSKV_WAIT_VM(2);
        else
            PSKV_WAIT_VM(0);
        __syncthreads();
        if (t + 5 <= T - 1)
            request(t + 5);
        if (t + 6 <= T - 1)
            request(t + 6);
    };

    unsigned long long bad_passes = 0; // bit n & 63: the workgroup's n-th pass has to be repeated
    int turn = 0;                      // number of the pass that comes next
    int p = blockIdx.x;
    PackedPass ps = packed_pass(a, p, npasses, nblocks, waves, wave);
    PackedBlock<STEPS> nxt = {0, 1, 0, 0, 1, 0u, 0u, 0u, 1u, false};
    unsigned q_off = 0;
    uintx4 q[8]; // this pass's Q fragments until their last use, then the next pass's
    // The next pass's block: its place in the list (z: where to look), its rows and Q.
    auto take_block = [&](const Args &a, const PackedArgs &pa, RowSearch z) __attribute__((always_inline)) {
        if (ps.active) {
            X.head = ps.head;
            const int r0 = ps.blk * kBlockRows;
            Walk w = find(a, pa, z, r0);
            PackedRow row;
            nxt = packed_block<STEPS>(a, pa, fresh_lane(X), w, r0, list, q_off, row, [&](int b) {
                return !list.even && b - z.cand < 64 ? __builtin_amdgcn_readlane(z.len, b - z.cand) : packed_len(a, b);
            });
        }
        load_q_packed(a, pa, fresh_lane(X), nxt.b, q_off, q);
    };
    RowSearch z = search_begin(a, ps.active ? ps.blk * kBlockRows : 0);
    take_block(a, pa, z);

    while (p < npasses) {
        // (the arguments are read again for every pass: kept over the passes, hundreds of scalars would be spilled to vector registers' lanes)
        const StreamPacked &call = first_parameter<StreamPacked>();
        const Args &a = call.a;
        const PackedArgs &pa = call.pa;
        if (!ps.exists) {
            ++turn;
            p += gridDim.x;
            ps = packed_pass(a, p, npasses, nblocks, waves, wave);
            z = search_begin(a, ps.active ? ps.blk * kBlockRows : 0);
            take_block(a, pa, z);
            continue;
        }
        set_vhead(a, X, ps.head);
        bool bad = false;
        const bool active = ps.active;
        const int pad_len = pair_len(a); // (asked for here: waited for together with the tiles)
        pass_top();
        if (!active) { // only staging
            for (int t = 2; t + 1 <= T - 2; t += 2)
                pair_top(t);
            p += gridDim.x;
            ps = packed_pass(a, p, npasses, nblocks, waves, wave);
            z = search_begin(a, ps.active ? ps.blk * kBlockRows : 0);
            take_block(a, pa, z);
        } else {
            const PackedBlock<STEPS> x = nxt;

            // ---- first prefix tile: scores, reference maximum ----
            floatx16 sA, sB; // raw scores of the current and of the next tile, roles alternating
#pragma unroll
            for (int e = 0; e < 16; ++e)
                sA[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
                sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*(lds_u128 *)(kimg(0) + ks * 1024)), as_bf16x8(q[ks]), sA,
                                                             0, 0, 0);
            Pre pre;
#pragma unroll
            for (int i = 0; i < kDist; ++i)
                pre.k[i] = *(lds_u128 *)(kimg(1) + i * 1024);
            float m = sA[0];
#pragma unroll
            for (int e = 1; e < 16; ++e)
                m = fmaxf(m, sA[e]);
            m = max_of_halves(m) * X.c; // (the other half-wave holds the other 16 keys)
            float l = 0.f;
            floatx16 o[4];
            uintx4 pA[2], pB[2]; // packed weights of the current and of the previous tile, roles alternating
            uintx4 skf[8], svf[2][4];

            // ---- pipeline over the prefix tiles (as above) ----
            pipe_tile<true, false, false, false, 0, true, true>(kimg(1), skf, vimg(0), kimg(2), vimg(0), pre, q, sA, sB,
                                                                X.c, m, 0, l, pA, pA, o);
            pipe_tile<true, false, true, true, 0, true, true>(kimg(2), skf, vimg(0), kimg(3), vimg(1), pre, q, sB, sA, X.c,
                                                              m, 0, l, pA, pB, o);
#define PSKV_STEP_PAIR(t)                                                                                              \
    do {                                                                                                               \
        pipe_tile<true, false, true, false, 0, true, true>(kimg((t) + 1), skf, vimg((t) - 1), kimg((t) + 2),           \
                                                           vimg(t), pre, q, sA, sB, X.c, m, 0, l, pB, pA, o);          \
        pipe_tile<true, false, true, false, 0, true, true>(kimg((t) + 2), skf, vimg(t),                                \
                                                           kimg((t) + 3 < T ? (t) + 3 : T - 1), vimg((t) + 1),         \
                                                           pre, q, sB, sA, X.c, m, 0, l, pA, pB, o);                   \
    } while (0)
            int t = 2;
            for (; t + 3 <= T - 2; t += 2) {
                pair_top(t);
                PSKV_STEP_PAIR(t);
            }
            // The last pair requests no further tiles; the window's K fragments and the lengths around the next pass's first row,
            // needed two or three steps from here, are requested now.
            const bool last_pair = t + 1 <= T - 2;
            if (last_pair)
                pair_top(t);
            p += gridDim.x;
            ps = packed_pass(a, p, npasses, nblocks, waves, wave);
            z = search_begin(a, ps.active ? ps.blk * kBlockRows : 0);
            load_window_k(pa, fresh_lane(X), x, 0, skf);
            if (last_pair) {
                PSKV_STEP_PAIR(t);
                t += 2;
            }
#undef PSKV_STEP_PAIR
            if (t <= T - 2) { // one step left over: do it and put scores and weights back in their places
                pipe_tile<true, false, true, false, 0, true, true>(kimg(t + 1), skf, vimg(t - 1), kimg(T - 1), vimg(t), pre,
                                                                   q, sA, sB, X.c, m, 0, l, pB, pA, o);
                sA = sB;
                pB[0] = pA[0];
                pB[1] = pA[1];
            }
            if (past) { // ragged last prefix tile: keys past the prefix are not visible
                int bits = (1 << (kTileKeys - past)) - 1;
                bits >>= 4 * fresh_lane(X).h; // element e holds key 8*(e/4) + e%4 + 4*h of the tile
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    sA[e] = hide_unless_bit(sA[e], bits, 8 * (e >> 2) + (e & 3));
            }
            load_window_v(pa, fresh_lane(X), x, 0, svf); // one step ahead of its use
            lds_u8 *const v_last = added_here(X.v_lane, ((T - 1) & (kRing - 1)) * kSlotBytes);
            // ---- last prefix tile: the "next scores" are the window's first ones ----
            pipe_tile<true, true, true, false, 0, false, true>(kimg(0), skf, added_here(X.v_lane, ((T - 2) & (kRing - 1)) * kSlotBytes), kimg(0), v_last, pre, q,
                                                               sA, sB, X.c, m, 0, l, pB, pA, o);

            // Unless the window goes on, Q has been used for the last time: the next pass's takes its place.
            const int head = X.head; // (of this pass)
            const bool more = STEPS > 1 && x.width > kTileKeys;
            if (!more)
                take_block(a, pa, z);

            // ---- first window step: mask and weights under the value product of the last prefix
            //      tile; then its own value product through the scratch tile ----
            pipe_tile<false, false, true, false, 2, false, false>(kimg(0), skf, v_last, kimg(0), vimg(0), pre, q, sB, sB,
                                                                  X.c, m, sees_bits(x, 0, fresh_lane(X).h), l, pA, pB, o);
            const Ctx Y = fresh_lane(X);
            if (more)
                load_window_k(pa, Y, x, kTileKeys, skf);
            pv_from_scratch(Y, svf[0], as_bf16x8(pB[0]), o);
            pv_from_scratch(Y, svf[1], as_bf16x8(pB[1]), o);
            if (more) {
                for (int k0 = kTileKeys;; k0 += kTileKeys) {
                    load_window_v(pa, fresh_lane(X), x, k0, svf);
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        sB[e] = 0.f;
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks)
                        sB = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(skf[ks]), as_bf16x8(q[ks]), sB, 0, 0, 0);
                    const bool again = STEPS > 2 && k0 + kTileKeys < x.width;
                    if (again)
                        load_window_k(pa, fresh_lane(X), x, k0 + kTileKeys, skf);
                    window_step_fixed(Y, sees_bits(x, k0, Y.h), sB, m, l, svf, o);
                    if (!again)
                        break;
                }
                take_block(a, pa, z);
            }

            bad = x.wide || __builtin_amdgcn_ballot_w64(!(l < kBig)) != 0;
            Ctx W = fresh_lane(X);
            W.head = head;
            store_packed(a, pa, W, x, list.align, m, l, o);
        }
        if (pair < pairs)
            store_pair(a, pa, pad_len);
        for (int n = 1; n < each && pair < pairs; ++n)
            store_pair(a, pa, pair_len(a));
        // the wavefront's verdict goes into the first word of its own scratch tile
        if (X.lane == 0)
            *(lds_int *)X.scr = bad ? 1 : 0;
        __syncthreads(); // ends the pass: the ring is free, the verdicts are visible
        if (__builtin_amdgcn_ballot_w64(*(lds_int *)(smem + kRing * kSlotBytes + (X.lane & (kNW - 1)) * kScrBytes) != 0))
            bad_passes |= 1ull << (turn & 63);
        ++turn;
    }
    while (pair < pairs)
        store_pair(a, pa, pair_len(a));

    // Rare: some row met scores far above its first tile's maximum, or a block's candidates lie far apart; what such a pass
    // stored is then replaced by the general path's result.  (Only such passes: one candidate in need of it among 300 x 40
    // positions, 40/40 heads, P 700: 320 us, all of a workgroup's passes 536, the general kernel 317.)
    if (bad_passes) {
        const StreamPacked &call = first_parameter<StreamPacked>();
        const Args &a = call.a;
        const PackedArgs &pa = call.pa;
        for (int p2 = blockIdx.x, n = 0; p2 < npasses; p2 += gridDim.x, ++n) {
            ps = packed_pass(a, p2, npasses, nblocks, waves, wave);
            if (!ps.exists || !(bad_passes >> (n & 63) & 1))
                continue;
            set_vhead(a, X, ps.head);
            GeneralBlock<STEPS> g;
            const int r0 = ps.active ? ps.blk * kBlockRows : 0;
            z = search_begin(a, r0);
            Walk w = find(a, pa, z, r0);
            packed_general_begin(a, pa, X, w, r0, list, g);
            uintx4 kv, vv;
            load_tile_chunks(a, X, ts, 0, kv, vv);
            __syncthreads(); // whatever the ring held has been used by every wavefront
            write_tile_chunks(X, ts, 0, smem, smem + kTileBytes, tid, kv, vv);
            __syncthreads();
            for (int kt = 0; kt < T; ++kt) {
                load_tile_chunks(a, X, ts, kt + 1 < T ? kt + 1 : kt, kv, vv);
                prefix_tile_classic(X, X.k_lane + (kt & 1) * kSlotBytes, X.v_lane + (kt & 1) * kSlotBytes, X.P - kt * kTileKeys, g.q, g.st);
                if (kt + 1 < T)
                    write_tile_chunks(X, ts, kt + 1, smem + ((kt + 1) & 1) * kSlotBytes, smem + ((kt + 1) & 1) * kSlotBytes + kTileBytes, tid, kv, vv);
                __syncthreads();
            }
            if (ps.active)
                packed_general_end(a, X, g);
        }
    }
}

// ------------------------------------------------------------------------------------------
// Candidate passes: suffix-side segments of several 32-key tiles (suffix, template tail and
// target together, Sec. 3.1).  Here the causal part is no longer a small correction after the
// prefix, and fetching a candidate's suffix K/V per wavefront, one exposed round trip per tile,
// dominates.  So a pass is cut out of ONE candidate: (candidate, KV head, group of up to 8 of the
// candidate's S*G/32 row blocks), and the ring simply goes on after the last prefix tile with
// the 32-key tiles of that candidate's own suffix K/V, up to the last key any row of the pass
// sees.  Every tile, prefix or suffix, is then staged once per pass by all 512 threads, several
// tiles ahead of its use, and every step is a step of the same three-stage pipeline; a step
// whose tile has keys some row does not see (ragged last prefix tile, suffix tiles at or past
// the row's own position) takes the masked form of the step, the limit being per row.
// A tile wholly in a row's future gives that row weights of exactly zero.
//
// Pass ids are laid out so that the groups of one (candidate, KV head) unit run at the same
// time on compute units of one XCD (workgroup ids go round the XCDs): the unit's suffix K/V is
// then fetched from HBM once and found in that XCD's L2 by the other groups.
// Preconditions (launcher): those of the pipelined passes above, and S*ks_stride_s*2 < 2^31.
// ------------------------------------------------------------------------------------------
struct CandShape {
    int nblk_c; // 32-row blocks per candidate (S*G/32, rounded up)
    int ngrp;   // passes per (candidate, KV head) unit
    int bpp;    // blocks per pass (the last pass of a unit may hold fewer)
};

struct CandPass {
    int vh, head, cand0; // as in Pass
    int b;               // candidate (global index)
    int cblk0, cblk_last; // first and last block of the pass within the candidate
    int blk;             // this wavefront's block in the instruction's row space (clamped)
    bool exists;         // the unit exists (unit ids are padded to a multiple of 8)
    bool active;         // the wavefront has a block
};

__device__ inline CandPass make_cand_pass(const Args &a, const CandShape &cs, int p, int npasses, int wave)
{
    CandPass ps;
    const int pc = p < npasses ? p : npasses - 1;
    const int q = pc >> 3, x = pc & 7;
    const int uq = q / cs.ngrp, grp = q - uq * cs.ngrp;
    const int units = a.B * a.Hkv;
    int u = uq * 8 + x;
    ps.exists = p < npasses && u < units;
    u = u < units ? u : units - 1;
    ps.b = u / a.Hkv;
    ps.head = u - ps.b * a.Hkv;
    const int n = ps.b / a.C;
    ps.vh = n * a.Hkv + ps.head;
    ps.cand0 = n * a.C;
    ps.cblk0 = grp * cs.bpp;
    const int rest = cs.nblk_c - ps.cblk0;
    const int nb = rest < cs.bpp ? rest : cs.bpp;
    ps.cblk_last = ps.cblk0 + nb - 1;
    ps.active = ps.exists && wave < nb;
    const int cblk = ps.cblk0 + wave;
    ps.blk = (ps.b - ps.cand0) * cs.nblk_c + (cblk < ps.cblk_last ? cblk : ps.cblk_last);
    return ps;
}

struct CandStager {
    const unsigned char *kp, *vp;       // prefix K and V of the pass's instruction and head
    const unsigned char *ks, *vs;       // suffix K and V of the pass's candidate and head
    unsigned k_off, v_off;              // prefix: this thread's chunk within a full tile, bytes
    unsigned k_off_last, v_off_last;    // ... within the last prefix tile (rows clamped into the prefix)
    unsigned tile_stride;               // bytes from one prefix tile to the next
    int k_row, v_row;                   // suffix: this thread's rows within a tile ...
    unsigned k_col, v_col, row_stride;  // ... byte offsets of its chunks within a row, bytes per row
    int Tp;                             // prefix tiles
    int last;                           // index of the pass's last tile, prefix and suffix tiles counted together
    int skmax;                          // last suffix key any row of the pass sees
};

// Tile kt of the pass (clamped to its last tile).  Suffix rows past skmax are fetched from row
// skmax: no valid row sees them, finite data is all that is needed.
__device__ inline void cand_stage_load(const CandStager &g, int kt, uintx4 &kv, uintx4 &vv)
{
    const int u = kt < g.last ? kt : g.last;
    if (u < g.Tp) {
        const unsigned base = (unsigned)u * g.tile_stride;
        const bool lastp = u == g.Tp - 1;
        kv = *reinterpret_cast<const uintx4 *>(g.kp + (base + (lastp ? g.k_off_last : g.k_off)));
        vv = *reinterpret_cast<const uintx4 *>(g.vp + (base + (lastp ? g.v_off_last : g.v_off)));
    } else {
        const int j0 = (u - g.Tp) * kTileKeys;
        const int kr = j0 + g.k_row < g.skmax ? j0 + g.k_row : g.skmax;
        const int vr = j0 + g.v_row < g.skmax ? j0 + g.v_row : g.skmax;
        kv = *reinterpret_cast<const uintx4 *>(g.ks + ((unsigned)kr * g.row_stride + g.k_col));
        vv = *reinterpret_cast<const uintx4 *>(g.vs + ((unsigned)vr * g.row_stride + g.v_col));
    }
}

// O^T += V^T P^T for one tile whose V image is in the ring.
__device__ inline void pv_tile(lds_u8 *v_img, const uintx4 (&pp)[2], floatx16 (&o)[4])
{
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
        o[ks & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_fragment(v_img, ks & 3, ks >> 2), as_bf16x8(pp[ks >> 2]),
                                                            o[ks & 3], 0, 0, 0);
}

template <bool WHOLE>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void stream_candidate_kernel(Args a, int npasses, CandShape cs)
{
    extern __shared__ __align__(16) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X = make_stream_ctx(a, smem, tid);
    const int rows_c = a.S * a.G; // rows of a candidate
    auto decode = [&](const CandPass &ps) __attribute__((always_inline)) {
        return decode_own<WHOLE>(a, X, ps.blk, ps.head, ps.cand0, ps.b - ps.cand0, cs.nblk_c);
    };
    // the block within its candidate, and the rows that exist from its first one on
    auto block_in_cand = [&](const CandPass &ps) { return ps.blk - (ps.b - ps.cand0) * cs.nblk_c; };
    auto block_rows = [&](const CandPass &ps) { return WHOLE ? kBlockRows : rows_c - block_in_cand(ps) * kBlockRows; };
    auto kimg = [&](int t) { return X.k_lane + (t & (kRing - 1)) * kSlotBytes; };
    auto vimg = [&](int t) { return X.v_lane + (t & (kRing - 1)) * kSlotBytes; };
    auto stage_write = [&](int kt, const uintx4 &kv, const uintx4 &vv) {
        lds_u8 *slot = smem + (kt & (kRing - 1)) * kSlotBytes + tid * 16;
        *(lds_u128 *)slot = kv;
        *(lds_u128 *)(slot + kTileBytes) = vv;
    };

    CandStager g;
    const TileSlot ts = make_tile_slot(tid);
    g.k_off = (unsigned)(ts.k_row * a.kp_sp + ts.k_chunk * 8) * 2u;
    g.v_off = (unsigned)(ts.v_row * a.kp_sp + ts.v_chunk * 8) * 2u;
    g.tile_stride = (unsigned)(kTileKeys * a.kp_sp) * 2u;
    g.k_row = ts.k_row;
    g.v_row = ts.v_row;
    g.k_col = (unsigned)ts.k_chunk * 16u;
    g.v_col = (unsigned)ts.v_chunk * 16u;
    g.row_stride = (unsigned)a.ks_ss * 2u;

    bool wg_bad = false, wg_short = false;
    int p = blockIdx.x;
    CandPass ps = make_cand_pass(a, cs, p, npasses, wave);
    BlockRows nxt = decode(ps);
    uintx4 q[8]; // this pass's Q fragments until their last use, then the next pass's
    load_q_block(a, X, nxt, q);

    while (p < npasses) {
        set_vhead(a, X, ps.vh);
        const int Tp = (X.P + kTileKeys - 1) / kTileKeys;
        const int len = len_uniform(a, ps.b);
        const int i_lo = (int)fdiv(ps.cblk0 * kBlockRows, a.div_g); // first suffix position of the pass
        const bool nothing = !ps.exists || i_lo >= len;             // no unit, or nothing but padding
        if (nothing || Tp < kMinTiles) {
            if (!nothing)
                wg_short = true; // prefix too short for the pipeline: left to the general sweep below
            else if (ps.active)
                store_zero_block_rows(a, X, nxt, block_rows(ps));
            p += gridDim.x;
            ps = make_cand_pass(a, cs, p, npasses, wave);
            nxt = decode(ps);
            load_q_block(a, X, nxt, q);
            continue;
        }
        const int i_hi = (int)fdiv(ps.cblk_last * kBlockRows + kBlockRows - 1, a.div_g);
        const int skmax = i_hi < len - 1 ? i_hi : len - 1;
        const int T = Tp + skmax / kTileKeys + 1;
        {
            const int nlast = X.P - (Tp - 1) * kTileKeys; // rows of the last prefix tile, 1..32
            const int kr = ts.k_row < nlast ? ts.k_row : nlast - 1, vr = ts.v_row < nlast ? ts.v_row : nlast - 1;
            g.k_off_last = (unsigned)(kr * a.kp_sp + ts.k_chunk * 8) * 2u;
            g.v_off_last = (unsigned)(vr * a.kp_sp + ts.v_chunk * 8) * 2u;
            g.Tp = Tp;
            g.last = T - 1;
            g.skmax = skmax;
            g.kp = reinterpret_cast<const unsigned char *>(X.kpg);
            g.vp = reinterpret_cast<const unsigned char *>(X.vpg);
            g.ks = reinterpret_cast<const unsigned char *>(X.ksg + (long long)ps.b * a.ks_sb);
            g.vs = reinterpret_cast<const unsigned char *>(X.vsg + (long long)ps.b * a.ks_sb);
        }
        const BlockRows row = nxt;
        // This wavefront's own share of the pass's tiles: the prefix and the suffix tiles up to the
        // last key its own block sees (Tw <= T); none at all if it has no block or its block holds
        // nothing but padding (then it only stores zeros).
        const int cblk = block_in_cand(ps), rows = block_rows(ps);
        const int i_lo_w = (int)fdiv(cblk * kBlockRows, a.div_g);
        const int i_hi_w = (int)fdiv(cblk * kBlockRows + kBlockRows - 1, a.div_g);
        const bool active = ps.active && i_lo_w < len;
        const int Tw = Tp + (i_hi_w < skmax ? i_hi_w : skmax) / kTileKeys + 1;
        const bool rvalid = active && row.ri < row.len;

        // The ring is free here (the barrier that ended the previous pass).  Tiles 0..3 go in at once.
        uintx4 kv0, vv0, kv1, vv1;
        {
            uintx4 kv2, vv2, kv3, vv3;
            cand_stage_load(g, 0, kv0, vv0);
            cand_stage_load(g, 1, kv1, vv1);
            cand_stage_load(g, 2, kv2, vv2);
            cand_stage_load(g, 3, kv3, vv3);
            stage_write(0, kv0, vv0);
            stage_write(1, kv1, vv1);
            stage_write(2, kv2, vv2);
            stage_write(3, kv3, vv3);
        }
        cand_stage_load(g, 4, kv0, vv0);
        cand_stage_load(g, 5, kv1, vv1);
        __syncthreads();

        // Visibility limit of tile t for this lane's row, as pipe_tile takes it: element e (key
        // offset 8*(e/4) + e%4 + 4*h within the tile) is visible iff its offset without the
        // 4*h is <= lim.  Prefix tiles are fully visible but for the end of a ragged last one;
        // suffix tile j holds keys 32*j.. of which the row sees those up to its own position.
        const int lim_suffix = row.ri - 4 * X.h + Tp * kTileKeys;
        const int lim_last_prefix = X.P - (Tp - 1) * kTileKeys - 1 - 4 * X.h;
        auto lim_of = [&](int t) { return t >= Tp ? lim_suffix - t * kTileKeys : (t == Tp - 1 ? lim_last_prefix : 1 << 20); };
        const int tm = X.P / kTileKeys; // first tile with keys that some row does not see (>= 2)

        // A wavefront without a block (the last pass of a unit may hold fewer than eight) takes part
        // in the staging and in the barriers only, and leaves the matrix cores of its SIMD to its
        // neighbour: same barriers, in the same order, as the path below.
        if (!active) {
            if (ps.active)
                store_zero_block_rows(a, X, row, rows);
            for (int t = 2; t + 1 <= T - 2; t += 2) {
                stage_write(t + 2, kv0, vv0);
                stage_write(t + 3, kv1, vv1);
                cand_stage_load(g, t + 4, kv0, vv0);
                cand_stage_load(g, t + 5, kv1, vv1);
                __syncthreads();
            }
            p += gridDim.x;
            ps = make_cand_pass(a, cs, p, npasses, wave);
            nxt = decode(ps);
            load_q_block(a, X, nxt, q);
            if (X.lane == 0)
                *(lds_int *)X.scr = 0;
            __syncthreads(); // ends the pass
            wg_bad |= __builtin_amdgcn_ballot_w64(*(lds_int *)(smem + kRing * kSlotBytes + (X.lane & (kNW - 1)) * kScrBytes) !=
                                                  0) != 0;
            continue;
        }

        // ---- first prefix tile: scores, reference maximum ----
        floatx16 sA, sB;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            sA[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*(lds_u128 *)(kimg(0) + ks * 1024)), as_bf16x8(q[ks]), sA,
                                                         0, 0, 0);
        Pre pre;
#pragma unroll
        for (int i = 0; i < kDist; ++i)
            pre.k[i] = *(lds_u128 *)(kimg(1) + i * 1024);
        float m = sA[0];
#pragma unroll
        for (int e = 1; e < 16; ++e)
            m = fmaxf(m, sA[e]);
        m = fmaxf(m, __shfl_xor(m, 32, 64)) * X.c;
        float l = 0.f;
        floatx16 o[4];
        uintx4 pA[2], pB[2];
        uintx4 nokf[8]; // stands in for the register K fragments no step here uses

        pipe_tile<true, false, false, false, false, true, true>(kimg(1), nokf, vimg(0), kimg(2), vimg(0), pre, q, sA, sB,
                                                                X.c, m, 0, l, pA, pA, o);
        pipe_tile<true, false, true, true, false, true, true>(kimg(2), nokf, vimg(0), kimg(3 < Tw ? 3 : Tw - 1), vimg(1), pre, q,
                                                              sB, sA, X.c, m, 0, l, pA, pB, o);
#define PSKV_CAND_PAIR(t, MASKED)                                                                                      \
    do {                                                                                                               \
        pipe_tile<true, false, true, false, MASKED, true, true>(kimg((t) + 1), nokf, vimg((t) - 1), kimg((t) + 2),     \
                                                                vimg(t), pre, q, sA, sB, X.c, m, lim_of(t), l, pB, pA, \
                                                                o);                                                    \
        pipe_tile<true, false, true, false, MASKED, true, true>(kimg((t) + 2), nokf, vimg(t),                          \
                                                                kimg((t) + 3 < Tw ? (t) + 3 : Tw - 1), vimg((t) + 1),  \
                                                                pre, q, sB, sA, X.c, m, lim_of((t) + 1), l, pA, pB,    \
                                                                o);                                                    \
    } while (0)
        int t = 2;
        for (; t + 1 <= Tw - 2 && t + 1 < tm; t += 2) { // pairs of fully visible tiles
            stage_write(t + 2, kv0, vv0);
            stage_write(t + 3, kv1, vv1);
            cand_stage_load(g, t + 4, kv0, vv0);
            cand_stage_load(g, t + 5, kv1, vv1);
            __syncthreads();
            PSKV_CAND_PAIR(t, false);
        }
        for (; t + 1 <= Tw - 2; t += 2) {
            stage_write(t + 2, kv0, vv0);
            stage_write(t + 3, kv1, vv1);
            cand_stage_load(g, t + 4, kv0, vv0);
            cand_stage_load(g, t + 5, kv1, vv1);
            __syncthreads();
            PSKV_CAND_PAIR(t, true);
        }
        const int t_own = t; // the wavefront's own tiles end here; staging for the others goes on below
#undef PSKV_CAND_PAIR
        if (t <= Tw - 2) { // one step left over: do it and put scores and weights back in their places
            pipe_tile<true, false, true, false, true, false, true>(kimg(t + 1), nokf, vimg(t - 1), kimg(Tw - 1), vimg(t), pre,
                                                                   q, sA, sB, X.c, m, lim_of(t), l, pB, pA, o);
            sA = sB;
            pB[0] = pA[0];
            pB[1] = pA[1];
        }

        // Q has been used for the last time: the next pass's Q takes its place
        p += gridDim.x;
        ps = make_cand_pass(a, cs, p, npasses, wave);
        nxt = decode(ps);
        load_q_block(a, X, nxt, q);

        // ---- last tile: its weights under the value product of the tile before, then its own ----
        pipe_tile<false, false, true, false, true, false, false>(kimg(0), nokf, vimg(Tw - 2), kimg(0), vimg(0), pre, q, sA, sA,
                                                                 X.c, m, lim_of(Tw - 1), l, pB, pA, o);
        pv_tile(vimg(Tw - 1), pA, o);

        const bool bad = __builtin_amdgcn_ballot_w64(rvalid && !(l < kBig)) != 0;
        // the rest of the pass's staging, for the wavefronts whose blocks see further (before this
        // wavefront's store: they are the ones the pass is waiting for)
        for (t = t_own; t + 1 <= T - 2; t += 2) {
            stage_write(t + 2, kv0, vv0);
            stage_write(t + 3, kv1, vv1);
            cand_stage_load(g, t + 4, kv0, vv0);
            cand_stage_load(g, t + 5, kv1, vv1);
            __syncthreads();
        }
        store_block_rows(a, X, row, m, l, o, rows);
        if (X.lane == 0)
            *(lds_int *)X.scr = bad ? 1 : 0;
        __syncthreads(); // ends the pass: the ring is free, the verdicts are visible
        wg_bad |= __builtin_amdgcn_ballot_w64(*(lds_int *)(smem + kRing * kSlotBytes + (X.lane & (kNW - 1)) * kScrBytes) !=
                                              0) != 0;
    }

    // The general sweep, as in the pipelined kernel above.
    if (wg_bad || wg_short)
        for (int p2 = blockIdx.x; p2 < npasses; p2 += gridDim.x) {
            const CandPass ps2 = make_cand_pass(a, cs, p2, npasses, wave);
            set_vhead(a, X, ps2.vh);
            if (ps2.exists && (wg_bad || (X.P + kTileKeys - 1) / kTileKeys < kMinTiles))
                general_pass(a, X, smem, tid, ps2.vh, WHOLE ? ps2.blk : block_in_cand(ps2), ps2.active, WHOLE ? 0 : ps2.b - ps2.cand0,
                             WHOLE ? 0 : rows_c);
        }
}

// ------------------------------------------------------------------------------------------
// Candidate passes of four blocks: workgroups of four wavefronts, two on a compute unit, so that one works while the
// other one waits for the first tiles of a pass, stores, or meets at the end of a pass - half of the time of a pass of
// eight, which nothing covers there.
//
// K and V have rings of their own, five tiles each, half images (pskv_mfma.hpp) filled by direct-to-LDS
// requests: 8 rows x 128 bytes each, 17 cycles of a compute unit where 32 rows x 32 bytes take 58, which at one
// request per 128 rows of queries instead of 256 would fill its address units.  Wavefronts 0 and 1
// fetch K (64 columns each), 2 and 3 V.  With s(t) the step of tile t, which reads K t+1 (and the beginning of t+2)
// and V t-1 (and the beginning of V t): barriers stand before the steps t = 1, 3, 5, ..., where everything requested before
// has landed.  Requested there, for the next pair: K t+4, t+5 - the slots of K t-1 and t, read before - and V t+2, t+3 -
// of V t-3 and t-2.  What the pair reads, K up to t+3 and V up to t+1, was requested a pair ago; tiles 0 .. 4 when the
// pass begins.
//
// What bounds it: instruction issue - a step is 16 matrix instructions and 64 vector ones, 32 more where
// the step masks - and the two wavefronts of a SIMD being served unevenly.  256 candidates x 128..160 positions, 28/4
// heads, P 128: 213 us in passes of eight, 197 us here; 300 x 96, 32/8, P 512: 388, 307.  (With a register spill in the steps
// 350: its reload waits for all requests in flight.  Hence the lane's places worked out by exclusive ors from two
// registers, and nothing else held that a step does not need.)
// ------------------------------------------------------------------------------------------
constexpr int kCW = 4;                          // wavefronts
constexpr int kCRing = 5;                       // tiles of K, and of V, in LDS
constexpr int kCLdsBytes = 2 * kCRing * kTileBytes; // half of a compute unit's

// pipe_tile with the images as half images (two per tile of K or V).  The lane's addresses in an image are
// worked out once, by the step that reads its first fragments, and handed on.
struct HalfPre {
    uintx4 k[kDist];
    bf16x8 v[kDist];
    unsigned ka[4], va[2][2]; // of the K image read next, of the V image read next
};
__device__ inline uintx4 k_frag(const unsigned (&at)[4], int i) { return *(lds_u128 *)(lds_at(at[i & 3]) + (i >> 2) * kHalfBytes); }
__device__ inline bf16x8 v_frag(const unsigned (&at)[2][2], int i)
{
    const int dt = i & 3, j = i >> 2;
    const int off = (dt >> 1) * kHalfBytes + j * 2048;
    short4v lo = lds_read_tr(lds_at(at[dt & 1][0]) + off), hi = lds_read_tr(lds_at(at[dt & 1][1]) + off + 1024);
    short8v v8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    bf16x8 f;
    __builtin_memcpy(&f, &v8, 16);
    return f;
}
__device__ inline void k_places(const HalfPlaces &hp, unsigned img, unsigned (&at)[4])
{
    unsigned first = hp.row + img;
    asm volatile("" : "+v"(first));
#pragma unroll
    for (int i = 0; i < 4; ++i)
        at[i] = first ^ (i << 5);
}
__device__ inline void v_places(const HalfPlaces &hp, unsigned img, unsigned (&at)[2][2])
{
    unsigned first = hp.col + img;
    asm volatile("" : "+v"(first));
#pragma unroll
    for (int i = 0; i < 4; ++i)
        at[i >> 1][i & 1] = first ^ ((i >> 1) << 6) ^ ((i & 1) << 7);
}
template <bool HAS_QK, bool HAS_PV, bool FRESH, bool MASK, bool NEXT_K, bool NEXT_V>
__device__ __attribute__((always_inline)) void pipe_half(const HalfPlaces &hp, unsigned k_after, unsigned v_cur, HalfPre &pre, const uintx4 (&q)[8],
                                                         const floatx16 &s, floatx16 &sn, float c, float m, int lim, float &l,
                                                         const uintx4 (&pp)[2], uintx4 (&pc)[2], floatx16 (&o)[4])
{
    uintx4 kfr[8];
    bf16x8 vfr[8];
    unsigned pk[8];
    float rs = 0.f;
    if (HAS_QK) {
#pragma unroll
        for (int e = 0; e < 16; ++e)
            sn[e] = 0.f;
#pragma unroll
        for (int i = 0; i < kDist; ++i)
            kfr[i] = pre.k[i];
    }
    if (HAS_PV) {
#pragma unroll
        for (int i = 0; i < kDist; ++i)
            vfr[i] = pre.v[i];
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        if (HAS_QK && ks + kDist < 8)
            kfr[ks + kDist] = k_frag(pre.ka, ks + kDist);
        if (HAS_PV && ks + kDist < 8)
            vfr[ks + kDist] = v_frag(pre.va, ks + kDist);
        if (NEXT_K && ks == 8 - kDist)
            k_places(hp, k_after, pre.ka);
        if (NEXT_V && ks == 8 - kDist)
            v_places(hp, v_cur, pre.va);
        if (NEXT_K && ks >= 8 - kDist)
            pre.k[ks - (8 - kDist)] = k_frag(pre.ka, ks - (8 - kDist));
        if (NEXT_V && ks >= 8 - kDist)
            pre.v[ks - (8 - kDist)] = v_frag(pre.va, ks - (8 - kDist));
        if (HAS_QK)
            sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kfr[ks]), as_bf16x8(q[ks]), sn, 0, 0, 0);
        if (HAS_PV) {
            floatx16 acc = o[ks & 3];
            if (FRESH && ks < 4) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    acc[e] = 0.f;
            }
            o[ks & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vfr[ks], as_bf16x8(pp[ks >> 2]), acc, 0, 0, 0);
        }
        float s0 = s[2 * ks], s1 = s[2 * ks + 1];
        if (MASK) {
            s0 = 8 * ((2 * ks) >> 2) + ((2 * ks) & 3) <= lim ? s0 : -INFINITY;
            s1 = 8 * ((2 * ks + 1) >> 2) + ((2 * ks + 1) & 3) <= lim ? s1 : -INFINITY;
        }
        const float p0 = fast_exp2(__builtin_fmaf(s0, c, -m));
        const float p1 = fast_exp2(__builtin_fmaf(s1, c, -m));
        pk[ks] = pack_bf16(p0, p1);
        rs += p0;
        rs += p1;
        asm volatile("" : "+v"(rs), "+v"(pk[ks]));
        __builtin_amdgcn_sched_barrier(0);
    }
    l += rs;
    pc[0] = uintx4{pk[0], pk[1], pk[2], pk[3]};
    pc[1] = uintx4{pk[4], pk[5], pk[6], pk[7]};
}

template <bool WHOLE>
__global__ __attribute__((amdgpu_flat_work_group_size(kCW * 64, kCW * 64), amdgpu_waves_per_eu(2, 2)))
void stream_candidate4_kernel(Args a, int npasses, CandShape cs)
{
    extern __shared__ __align__(256) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X = make_stream_ctx(a, smem, tid);
    X.scr = smem + wave * kScrBytes; // (in the ring of K, which is free when a block is stored)
    const HalfPlaces hp = half_places(X.lane);
    const int rows_c = a.S * a.G; // rows of a candidate
    auto decode = [&](const CandPass &ps) __attribute__((always_inline)) {
        return decode_own<WHOLE>(a, X, ps.blk, ps.head, ps.cand0, ps.b - ps.cand0, cs.nblk_c);
    };
    auto block_in_cand = [&](const CandPass &ps) { return ps.blk - (ps.b - ps.cand0) * cs.nblk_c; };
    auto block_rows = [&](const CandPass &ps) { return WHOLE ? kBlockRows : rows_c - block_in_cand(ps) * kBlockRows; };
    const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_addr(smem));
    auto kimg = [&](int t) { return lds0 + ((unsigned)t % kCRing) * kTileBytes; };
    auto vimg = [&](int t) { return lds0 + (kCRing + (unsigned)t % kCRing) * kTileBytes; };

    // Staging: this wavefront's image of a tile (K or V, columns 0..63 or 64..127), four pieces of 8 rows x 128 bytes, as half_put
    // would put them: the lane's row and 16-byte chunk in even and in odd pieces.
    auto row_of = [&](int lane, int g) { return ((unsigned)lane >> 3) ^ (g & 1); };
    auto col_of = [&](int lane, int g) { return ((((unsigned)lane & 7u) ^ half_swz(row_of(lane, g))) << 4) + 128u * (wave & 1); };
    lds_u8 *const ring = smem + (wave < 2 ? 0 : kCRing * kTileBytes) + (wave & 1) * kHalfBytes;
    const unsigned pre_stride = (unsigned)a.kp_sp * 2u, own_stride = (unsigned)a.ks_ss * 2u; // bytes per row
    const unsigned pre_e = row_of(X.lane, 0) * pre_stride + col_of(X.lane, 0), pre_o = row_of(X.lane, 1) * pre_stride + col_of(X.lane, 1);
    const unsigned own_e = row_of(X.lane, 0) * own_stride + col_of(X.lane, 0), own_o = row_of(X.lane, 1) * own_stride + col_of(X.lane, 1);

    bool bad = false, wg_short = false;
    int p = blockIdx.x;
    CandPass ps = make_cand_pass(a, cs, p, npasses, wave);
    BlockRows nxt = decode(ps);
    uintx4 q[8]; // this pass's Q fragments until their last use, then the next pass's
    load_q_block(a, X, nxt, q);

    while (p < npasses) {
        set_vhead(a, X, ps.vh);
        const int Tp = (X.P + kTileKeys - 1) / kTileKeys;
        const int len = len_uniform(a, ps.b);
        const int i_lo = (int)fdiv(ps.cblk0 * kBlockRows, a.div_g); // first suffix position of the pass
        const bool nothing = !ps.exists || i_lo >= len;             // no unit, or nothing but padding
        if (nothing || Tp < kMinTiles) {
            if (!nothing)
                wg_short = true; // prefix too short for the pipeline: left to the general sweep below
            else if (ps.active)
                store_zero_block_rows(a, X, nxt, block_rows(ps));
            p += gridDim.x;
            ps = make_cand_pass(a, cs, p, npasses, wave);
            nxt = decode(ps);
            load_q_block(a, X, nxt, q);
            continue;
        }
        const int i_hi = (int)fdiv(ps.cblk_last * kBlockRows + kBlockRows - 1, a.div_g);
        const int skmax = i_hi < len - 1 ? i_hi : len - 1;
        const int T = Tp + skmax / kTileKeys + 1;
        const unsigned char *const pre_base = reinterpret_cast<const unsigned char *>(wave < 2 ? X.kpg : X.vpg);
        const unsigned char *const own_base = reinterpret_cast<const unsigned char *>(wave < 2 ? X.ksg : X.vsg) + (long long)ps.b * a.ks_sb * 2;
        auto request = [&](int u) { // this wavefront's part of tile u
            const bool own = u >= Tp;
            const unsigned stride = own ? own_stride : pre_stride;
            const int first = (own ? u - Tp : u) * kTileKeys, last = own ? skmax : X.P - 1;
            const unsigned char *base = own ? own_base : pre_base;
            lds_u8 *img = ring + ((unsigned)u % kCRing) * kTileBytes;
            if (first + kTileKeys - 1 <= last) {
                base += (unsigned long long)(unsigned)first * stride;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    request_to_lds(base, own ? (g & 1 ? own_o : own_e) : (g & 1 ? pre_o : pre_e), img + g * 1024);
                    base += 8 * stride;
                }
            } else { // (the last row stands in for those behind it: never visible)
                int lane = X.lane;
                asm volatile("" : "+v"(lane)); // (nothing of this is held across the steps)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int row = first + 8 * g + (int)row_of(lane, g);
                    request_to_lds(base, (unsigned)(row < last ? row : last) * stride + col_of(lane, g), img + g * 1024);
                }
            }
        };
        const BlockRows row = nxt;
        const int cblk = block_in_cand(ps), rows = block_rows(ps);
        const int i_lo_w = (int)fdiv(cblk * kBlockRows, a.div_g);
        const int i_hi_w = (int)fdiv(cblk * kBlockRows + kBlockRows - 1, a.div_g);
        const bool active = ps.active && i_lo_w < len;
        const int Tw = Tp + (i_hi_w < skmax ? i_hi_w : skmax) / kTileKeys + 1;
        const bool rvalid = active && row.ri < row.len;

        // The rings are free here (the barrier that ended the previous pass).
#pragma unroll
        for (int u = 0; u < kCRing; ++u)
            if (u < T)
                request(u);
        if (T >= kCRing)
            PSKV_WAIT_VM(8);
        else
            PSKV_WAIT_VM(0);
        __syncthreads();
        auto top = [&](int t) { // of the steps t and t+1, t odd
            PSKV_WAIT_VM(0);
            __syncthreads();
            const int u = wave < 2 ? t + 4 : t + 2;
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (u + i >= kCRing && u + i <= T - 1)
                    request(u + i);
        };

        const int lim_suffix = row.ri - 4 * X.h + Tp * kTileKeys;
        const int lim_last_prefix = X.P - (Tp - 1) * kTileKeys - 1 - 4 * X.h;
        auto lim_of = [&](int t) { return t >= Tp ? lim_suffix - t * kTileKeys : (t == Tp - 1 ? lim_last_prefix : 1 << 20); };
        const int tm = X.P / kTileKeys; // first tile with keys that some row does not see (>= 2)

        if (!active) { // takes part in the staging and in the barriers only
            for (int t = 1; t <= T - 1; t += 2)
                top(t);
            if (ps.active)
                store_zero_block_rows(a, X, row, rows);
            p += gridDim.x;
            ps = make_cand_pass(a, cs, p, npasses, wave);
            nxt = decode(ps);
            load_q_block(a, X, nxt, q);
            __syncthreads(); // ends the pass
            continue;
        }
        float l = 0.f;
        floatx16 o[4];
        floatx16 sA, sB;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            sA[e] = 0.f;
        HalfPre pre;
        k_places(hp, kimg(0), pre.ka);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            sA = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(k_frag(pre.ka, ks)), as_bf16x8(q[ks]), sA, 0, 0, 0);
        k_places(hp, kimg(1), pre.ka);
#pragma unroll
        for (int i = 0; i < kDist; ++i)
            pre.k[i] = k_frag(pre.ka, i);
        float m = sA[0];
#pragma unroll
        for (int e = 1; e < 16; ++e)
            m = fmaxf(m, sA[e]);
        m = fmaxf(m, __shfl_xor(m, 32, 64)) * X.c;
        uintx4 pA[2], pB[2];
        pipe_half<true, false, false, false, true, true>(hp, kimg(2), vimg(0), pre, q, sA, sB, X.c, m, 0, l, pA, pA, o);
#define PSKV_CAND4_PAIR(FRESH, MASK1, MASK2)                                                                                  \
    do {                                                                                                                     \
        top(t);                                                                                                              \
        pipe_half<true, true, FRESH, MASK1, true, true>(hp, kimg(t + 2), vimg(t), pre, q, sB, sA, X.c, m, lim_of(t), l, pA, \
                                                         pB, o);                                                             \
        pipe_half<true, true, false, MASK2, true, true>(hp, kimg(t + 3 < Tw ? t + 3 : Tw - 1), vimg(t + 1), pre, q, sA, sB, \
                                                         X.c, m, lim_of(t + 1), l, pB, pA, o);                               \
    } while (0)
        int t = 1;
        PSKV_CAND4_PAIR(true, false, true); // (tile 2 may be the prefix's ragged last one)
        t = 3;
        for (; t + 1 <= Tw - 2 && t + 1 < tm; t += 2)
            PSKV_CAND4_PAIR(false, false, false);
        for (; t + 1 <= Tw - 2; t += 2)
            PSKV_CAND4_PAIR(false, true, true);
#undef PSKV_CAND4_PAIR
        top(t); // (t: Tw - 2 or Tw - 1, in either case the last pair's first step)
        if (t <= Tw - 2) {
            pipe_half<true, true, false, true, false, true>(hp, 0, vimg(t), pre, q, sB, sA, X.c, m, lim_of(t), l, pA, pB, o);
            sB = sA;
            pA[0] = pB[0];
            pA[1] = pB[1];
            ++t;
        }
        // Q has been used for the last time: the next pass's Q takes its place
        p += gridDim.x;
        ps = make_cand_pass(a, cs, p, npasses, wave);
        nxt = decode(ps);
        load_q_block(a, X, nxt, q);
        // ---- last tile: its weights under the value product of the tile before, then its own ----
        pipe_half<false, true, false, true, false, false>(hp, 0, 0, pre, q, sB, sB, X.c, m, lim_of(Tw - 1), l, pA, pB, o);
        v_places(hp, vimg(Tw - 1), pre.va);
#pragma unroll
        for (int i = 0; i < 8; ++i)
            o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_frag(pre.va, i), as_bf16x8(pB[i >> 2]), o[i & 3], 0, 0, 0);
        // staging for the wavefronts whose blocks see further (before this wavefront's store: they are the ones the pass
        // is waiting for)
        for (t = Tw | 1; t <= T - 1; t += 2)
            top(t);
        // (the slots of K that tiles T and T + 1 would take: nobody reads there any more)
        X.scr = smem + ((unsigned)(T + (wave >> 1)) % kCRing) * kTileBytes + (wave & 1) * kScrBytes;
        bad |= __builtin_amdgcn_ballot_w64(rvalid && !(l < kBig)) != 0;
        store_block_rows(a, X, row, m, l, o, rows);
        __syncthreads(); // ends the pass: the rings are free
    }

    // The general sweep, as in the pipelined kernel above.
    if (X.lane == 0)
        *(lds_int *)(smem + wave * 4) = bad ? 1 : 0;
    __syncthreads();
    const bool wg_bad = __builtin_amdgcn_ballot_w64(*(lds_int *)(smem + (X.lane & (kCW - 1)) * 4) != 0) != 0;
    __syncthreads();
    if (wg_bad || wg_short) {
        X.scr = smem + 2 * kSlotBytes + wave * kScrBytes;
        for (int p2 = blockIdx.x; p2 < npasses; p2 += gridDim.x) {
            const CandPass ps2 = make_cand_pass(a, cs, p2, npasses, wave);
            set_vhead(a, X, ps2.vh);
            if (ps2.exists && (wg_bad || (X.P + kTileKeys - 1) / kTileKeys < kMinTiles))
                general_pass<kCW * 64>(a, X, smem, tid, ps2.vh, WHOLE ? ps2.blk : block_in_cand(ps2), ps2.active, WHOLE ? 0 : ps2.b - ps2.cand0,
                                       WHOLE ? 0 : rows_c);
        }
    }
}

int device_cu_count(hipError_t &e)
{
    static DeviceSlots cu_by_device;
    return device_setup_once(cu_by_device, e, [] {
        hipError_t s = hipFuncSetAttribute(reinterpret_cast<const void *>(stream_general_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        for (auto kernel : {stream_pipelined_kernel<true, true>, stream_pipelined_kernel<true, false>, stream_pipelined_kernel<false, true>,
                            stream_pipelined_kernel<false, false>})
            if (s == hipSuccess)
                s = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        for (auto kernel : {stream_packed_kernel<1>, stream_packed_kernel<2>, stream_packed_kernel<3>})
            if (s == hipSuccess)
                s = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        for (auto kernel : {stream_candidate4_kernel<true>, stream_candidate4_kernel<false>})
            if (s == hipSuccess)
                s = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kCLdsBytes);
        for (auto kernel : {stream_candidate_kernel<true>, stream_candidate_kernel<false>})
            if (s == hipSuccess)
                s = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        return s;
    });
}

// Whether the pipelined kernels' blocks, each inside one candidate, are the better ones: see launch_resident.
bool own_blocks_fit(const Args &a)
{
    const long long rows_c = (long long)a.S * a.G, nb = (rows_c + kBlockRows - 1) / kBlockRows;
    return rows_c * 16 >= nb * kBlockRows * 13 && a.C * nb <= 0x7fffffffLL / kBlockRows - kNW && stream_pass_ids(a, a.C * nb) <= 0x7fffffffLL - 8;
}

// The candidate passes that take a problem, if any: the one place where this is decided.
enum class CandPasses { none, four, eight };
CandPasses candidate_passes(const Args &a, int num_cu)
{
    const int max_tiles = (a.P + kTileKeys - 1) / kTileKeys;
    const long long rows_c = (long long)a.S * a.G, nb = (rows_c + kBlockRows - 1) / kBlockRows; // rows and own blocks of a candidate
    if (a.S <= kTileKeys || max_tiles < kMinTiles || (long long)a.P * a.kp_sp * 2 >= 0x7fffffffLL || (long long)a.S * a.ks_ss * 2 >= 0x7fffffffLL ||
        !own_blocks_fit(a) || !block_offsets_fit(a))
        return CandPasses::none;
    const bool whole = rows_c % kBlockRows == 0, resident = resident_supported(a);
    auto rounds = [&](long long passes) { return (passes + num_cu - 1) / num_cu; };
    const long long units = ((long long)a.B * a.Hkv + 7) / 8 * 8, ngrp8 = (nb + kNW - 1) / kNW, ngrp4 = (nb + kCW - 1) / kCW;
    const long long r8 = rounds(units * ngrp8), r4 = rounds(units * ngrp4); // passes per compute unit
    const bool fit8 = units * ngrp8 <= 0x7fffffffLL - 8, fit4 = units * ngrp4 <= 0x7fffffffLL - 2 * num_cu;

    // Passes of eight, only where a compute unit takes twice as many passes of four: they fetch the tiles half as often, which
    // long prefixes gain by.  us, of eight and of four, 32/8 heads (what a compute unit takes of either): 300 candidates: P 1500: 128
    // positions (19, 38): 924, 960; 64 (10, 19): 474, 458; 96 (19, 29): 869, 711; P 512: 104 (19, 38): 386, 400; 64: 205,
    // 190; 96: 388, 307; 24 candidates x 64 (1, 2): P 1500: 44.8, 46.4.
    // Resident prefixes: no difference on the whole (P 128: 300 x 120 (19, 38): 209, 218; 60 x 48..64 (2, 4): 23.0, 21.1; P 200:
    // 300 x 120: 271, 260; P 256: 60 x 120 (4, 8): 55.5, 57.2), but of three tiles (P 78: 220 x 115 (14, 28): 162, 143; P 79: 122 x
    // 21..40: 35, 30; P 94: 14 x 77 (1, 2): 12.3, 11.0).
    bool eight = fit8 && r4 >= 2 * r8 && nb * 10 >= ngrp8 * kNW * 6 && !(resident && max_tiles == kMinTiles);

    if (resident && !whole) {
        // Against the resident general kernel, whose wavefronts have `each` blocks and take the own steps one by one.
        const long long each = resident_split(a, (a.C * rows_c + kBlockRows - 1) / kBlockRows, kNW, num_cu).each;
        const bool many = a.S > 4 * kTileKeys;
        // Passes of eight, two thirds full and more: as many as blocks, one and a half times with more than four own steps.  us,
        // general kernel and passes of eight (`each`, passes per compute unit): P 99: 12 candidates x 87 positions (32/8 heads; 1, 1):
        // 16.9, 13.0; P 151: 20 x 132 (32/8; 2, 2): 30.3, 25.2; beyond: P 169: 49 x 74 (32/4; 2, 3): 30.2, 33.0; P 145: 247 x 22..45
        // (32/8; 6, 8): 64, 76; P 164: 161 x 113 (32/4; 9, 11): 136, 142; more own steps: P 222: 37 x 158 (28/4; 3, 3): 56, 45.
        // Passes of four, three quarters full and more: up to 9 for 4 blocks, 3 for 1 with more than four own steps.  us, general
        // kernel and passes of four (`each`, passes per compute unit): P 213: 10 x 69 (32/8; 1, 1): 17.8, 11.1; P 70: 35 x 56..66 (32/4;
        // 2, 3): 22.1, 15.6; P 189: 28 x 26..38 (32/4; 1, 2): 15.6, 12.6; P 169: 49 x 74 (32/4; 2, 4): 30.2, 26.6; P 162: 199 x 53
        // (28/4; 5, 10): 56.9, 57.5; beyond: P 227: 237 x 65 (32/4; 8, 19): 117, 119; P 164: 161 x 113 (32/4; 9, 21): 136, 139; P 242:
        // 116 x 70 (32/4; 4, 10): 57, 61; P 206: 203 x 41 (28/4; 4, 10): 51, 55; P 171: 198 x 58 (28/4; 5, 13): 59, 68; more own
        // steps: P 77: 13 x 135 (32/8; 1, 3): 20.1, 16.9; five eighths full: P 78: 97 x 159 (40/40; 11, 31): 221, 165; P 168: 265 x 58..157
        // (32/32; 28, 83): 448, 512; P 157: 48 x 60..151 (32/32; 4, 12): 66, 73; P 126: 37 x 130 (32/32; 3, 10): 48, 54.
        // Prefixes of their own lengths may be too short for these passes, which then sweep them on the general path: where the longest has
        // three or four tiles, up to 7 and 8 for 4.  us, real prefixes a third of P and more: P 93: 264 x 87 (40/40, eight instructions;
        // 24, 42): 376, 292; P 116: 20 x 148 (32/8, two; 2, 4): 33.7, 22.6 (passes of eight); beyond:
        // P 86: 112 x 77 (32/8, two; 5, 11): 49.5, 57.7; P 69: 48 x 85..123 (32/8, two; 3, 6): 35.5, 47.1; P 115: 222 x 46..52 (28/4,
        // two; 5, 11): 55.2, 67.8.
        const int most = a.plen && max_tiles <= kMinTiles + 1 ? max_tiles + 4 : many ? 12 : 9; // passes for 4 blocks
        if (nb * 4 < ngrp4 * kCW * 3 || r4 * 4 > most * each)
            return CandPasses::none;
        eight = eight && nb * 3 >= ngrp8 * kNW * 2 && r8 * 2 <= each * (many ? 3 : 2);
        return eight ? CandPasses::eight : fit4 ? CandPasses::four : CandPasses::none;
    }
    // Against the pipelined passes, whose blocks fetch their own keys by themselves and lose some three tiles' time to them.
    // us, pipelined passes and passes of four (rounds of the chip; passes of four per compute unit): 250 candidates, P 600: 128
    // positions, 32/32 heads (16, 32): 508, 427; 96 (12, 32): 358, 389; 72, 32/8 (9, 24): 221, 246; P 1500: 39 x 28/4 (5, 12): 239,
    // 263; P 128: 215, 177; 64 candidates, P 1500, 39 x 28/4 (2, 3): 87, 70; 300 x 40, 32/8, P 512 (6, 19): 121, 153; 181 x 88,
    // 32/8, P 1750 (8, 17): 441, 474; at the line: 70 x 133, 32/8, P 834 (5, 11): 175, 160; just beyond: P 300: 250 x 96, 32/32 (12, 32):
    // 263, 249; P 834: 100 x 133, 32/8 (7, 16): 250, 242.
    // Long prefixes and rows that fill no whole number of blocks: against the general passes as well, as long as there are hardly more of
    // the others and up to 1024 prefix rows.  us, general passes and passes of eight (rounds of the chip): 64 x 109 (32/8, P 464;
    // 4, 4): 121, 84; 50 x 148 (32/8, P 424; 4, 5): 105, 81; 12 x 156 (32/32, P 2018; 1, 2): 84, 103; 245 x 34 (32/8, P 676; 5, 8):
    // 169, 161 (pipelined passes 131).
    const long long rp = rounds(stream_pass_ids(a, a.C * nb)), full_rounds = rounds(stream_pass_ids(a));
    const bool any = whole || resident, full8 = fit8 && nb * 10 >= ngrp8 * kNW * 6 && (any || r8 * 7 <= full_rounds * 10);
    if (eight && full8)
        return CandPasses::eight;
    return fit4 && r4 * max_tiles <= 2 * rp * (max_tiles + 3) && (any || full8 || (r4 * 10 <= full_rounds * 22 && a.P <= 1024)) ? CandPasses::four
                                                                                                                            : CandPasses::none;
}

} // namespace

bool mfma_supported(const Args &a, int dtype)
{
    if (dtype != 1 || a.D != kD)
        return false;
    const long long rows = (long long)a.C * a.S * a.G;
    return rows <= 0x7fffffffLL - kPassRows && stream_pass_ids(a) <= 0x7fffffffLL - 8;
}

hipError_t launch_mfma(const Args &a, hipStream_t stream)
{
    if (!resident_supported(a))
        return launch_stream(a, stream);
    // Suffix-side segments longer than one 32-key step (suffix, template and target together,
    // Sec. 3) go to the streamed kernels, which run every suffix step against the fixed reference, where
    // the resident kernels would fall back to their general path for such shapes: all that fill
    // whole blocks of rows, and of the others those that the candidate passes are better at.
    const int max_tiles = (a.P + kTileKeys - 1) / kTileKeys;
    bool long_suffix = a.S > kTileKeys && max_tiles >= kMinTiles && (long long)a.P * a.kp_sp * 2 < 0x7fffffffLL;
    if (long_suffix && (long long)a.S * a.G % kBlockRows != 0) {
        hipError_t e;
        const int num_cu = device_cu_count(e);
        if (e != hipSuccess)
            return e;
        long_suffix = candidate_passes(a, num_cu) != CandPasses::none;
    }
    return long_suffix ? launch_stream(a, stream) : launch_resident(a, stream);
}

hipError_t launch_stream(const Args &a, hipStream_t stream)
{
    hipError_t e;
    const int num_cu = device_cu_count(e);
    if (e != hipSuccess)
        return e;
    const int max_tiles = (a.P + kTileKeys - 1) / kTileKeys;
    const long long rows_c = (long long)a.S * a.G, nb = (rows_c + kBlockRows - 1) / kBlockRows; // rows and own blocks of a candidate
    const bool whole = rows_c % kBlockRows == 0;
    bool pipelined = own_blocks_fit(a) && max_tiles >= kMinTiles && (long long)a.P * a.kp_sp * 2 < 0x7fffffffLL && block_offsets_fit(a);
    auto rounds = [&](long long passes) { return (passes + num_cu - 1) / num_cu; };
    const long long full_rounds = rounds(stream_pass_ids(a));
    // Long suffix-side segments: candidate passes of eight blocks, or of four, two at a time on a compute unit.
    if (const CandPasses passes = candidate_passes(a, num_cu); passes != CandPasses::none) {
        const bool eight = passes == CandPasses::eight;
        const int waves = eight ? kNW : kCW;
        const CandShape cs = {(int)nb, (int)((nb + waves - 1) / waves), nb < waves ? (int)nb : waves};
        const long long npasses = ((long long)a.B * a.Hkv + 7) / 8 * 8 * cs.ngrp, places = eight ? num_cu : 2 * num_cu;
        auto kernel = eight ? (whole ? stream_candidate_kernel<true> : stream_candidate_kernel<false>)
                            : (whole ? stream_candidate4_kernel<true> : stream_candidate4_kernel<false>);
        return launch_kernel(kernel, dim3((unsigned)(npasses < places ? npasses : places)), dim3(waves * 64), eight ? kLdsBytes : kCLdsBytes, stream,
                             a, (int)npasses, cs);
    }
    // Rows packed by their lengths, where there are lengths.  us, in the kernels below and so: 300 candidates, P 700: 16 positions, 40/40 heads: 118, 100;
    // 20..40: 298, 201; 12..24, 28/4: 96, 80; 700, P 300, 40/40: 40: 469, 366; 64: 555, 555; 32..64: 498, 463; 16 x 24, P 700: 35.0, 19.9.
    // Not whole blocks of grouped heads or of one block per candidate: which is faster depends on lengths that the host does not know, and
    // without padding the pipelined kernel is: 1500 x 32, 32/8, P 400: 423, 442 (16..32: 404, 350); 256 x 32, P 2048: 241, 245 (233, 186);
    // 300 x 32, 40/40, P 700: 178, 194 (170, 171).  What this costs: 2 to 5 % where nothing is padded and own blocks are nearly full (300 x 24, 28/4, P 700: 97,
    // 101; 300 x 28, 40/40: 173, 182; 120 x 24, 28/4, P 512: 37.8, 38.6, but at 12..24 of them 36.9, 25.3), and calls of two rounds of the chip that stay two: 40 x
    // 32..64, 40/40, P 1000: 76, 83.  Choosing whole candidates' blocks there by counting rounds on the device gave 77.5, and cost every call half a us.
    if (PackedArgs pa; a.len && a.Np == 1 && (!whole || (a.G == 1 && a.S > kTileKeys)) && max_tiles >= kMinTiles && a.S <= 2 * kTileKeys && (long long)a.P * a.kp_sp * 2 < 0x7fffffffLL &&
                       a.C * nb <= 0x7fffffffLL / kBlockRows && (long long)a.C * a.Hkv < 0x7fffffffLL - num_cu * kNW &&
                       stream_pass_ids(a, a.C * nb) <= 0x7fffffffLL - 8 && packed_args(a, (unsigned)num_cu, kNW, pa)) {
        const int steps = packed_steps(a, 3, pa.dense);
        auto kernel = steps == 1 ? stream_packed_kernel<1> : steps == 2 ? stream_packed_kernel<2> : stream_packed_kernel<3>;
        return launch_kernel(kernel, dim3((unsigned)num_cu), dim3(kNW * 64), kLdsBytes, stream, StreamPacked{a, pa});
    }
    // Own blocks make more passes, each in 0.7 of the general kernel's time, 0.8 with the second own step: not where
    // that costs a round of the chip.
    // us, general and pipelined: 512 candidates x 29 positions (32/32 heads, P 512): 252, 189; 512 x 26: 221, 178; 1024
    // x 30 (32/8): 388, 313; 300 x 13 (32/8, P 700; 2 rounds, 3 rounds): 66, 69; 43 x 113 (40/40, P 603; 3, 4): 109, 113.
    if (pipelined && !whole)
        pipelined = rounds(stream_pass_ids(a, a.C * nb)) * (a.S <= kTileKeys ? 7 : 8) <= full_rounds * 10;
    const long long npasses = pipelined ? stream_pass_ids(a, a.C * nb) : stream_pass_ids(a);
    const unsigned grid = (unsigned)(npasses < num_cu ? npasses : num_cu);
    if (!pipelined)
        return launch_kernel(stream_general_kernel, dim3(grid), dim3(kNW * 64), kLdsBytes, stream, a, (int)npasses);
    auto kernel = a.S <= kTileKeys ? (whole ? stream_pipelined_kernel<true, true> : stream_pipelined_kernel<true, false>)
                                   : (whole ? stream_pipelined_kernel<false, true> : stream_pipelined_kernel<false, false>);
    return launch_kernel(kernel, dim3(grid), dim3(kNW * 64), kLdsBytes, stream, a, (int)npasses, (int)nb, make_fastdiv((unsigned)nb));
}

} // namespace pskv
