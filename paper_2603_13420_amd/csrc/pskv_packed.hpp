// Packed rows: the valid query rows of one (instruction, KV head) pair, candidate by candidate, each candidate's rows
// (row i*G + g of position i and head g of the group) filled up to a multiple of `align`:
//   1   nothing between candidates, blocks of 32 rows whatever candidates they belong to, so that no matrix work is
//       spent on padding (a seventh of the blocks with lengths of 16..24 of 24 and four heads in a group, three eighths with 20 rows of 32);
//   32  every block inside one candidate, which has as many as its valid rows need.
// The keys that a block's rows see besides the prefix lie in one WINDOW, the positions of the block's candidates
// from the first one's first to the last row's own, and a row sees those from its candidate's first one to itself.
//
// A list whose runs are all a full candidate's is `even`: places in it are a division away, and its blocks can go to the wavefronts in turn.
//
// The lengths are in device memory.  Every workgroup adds them up (`PackedList`), finds the candidate of the row it begins
// with and goes on from candidate to candidate (`Walk`).
#pragma once
#include "pskv_mfma.hpp"

namespace pskv {

// What a kernel over packed rows is given besides the problem.  Strides in bytes.
struct PackedArgs {
    unsigned q_sb, q_ss, q_sh, o_sb, o_ss, o_sh, k_sb, k_ss;
    int span;       // candidates of one block at most, counted from its first one, for which 32-bit offsets from that one's rows reach
    bool dense;     // windows of align 1 fit the kernel's
    FastDiv div_n;  // division by the number of workgroups that share a list
    FastDiv div_w;  // ... of wavefronts
    FastDiv div_run; // by the rows of a full candidate, filled up to whole blocks
};

// False: a stride is too long for the 24-bit multiplications of the offsets (16 MB), or a candidate for 32-bit ones.
inline bool packed_args(const Args &a, unsigned sharers, int waves, PackedArgs &x)
{
    const long long strides[] = {a.q_sb, a.q_ss, a.q_sh, a.o_sb, a.o_ss, a.o_sh, a.ks_sb, a.ks_ss};
    long long sb = 1;
    for (const long long s : strides) {
        if (s < 0 || s * 2 >= 1 << 24)
            return false;
        sb = s > sb ? s : sb;
    }
    if (!block_offsets_fit(a) || a.S > 2 * 32)
        return false;
    x.q_sb = (unsigned)a.q_sb * 2, x.q_ss = (unsigned)a.q_ss * 2, x.q_sh = (unsigned)a.q_sh * 2;
    x.o_sb = (unsigned)a.o_sb * 2, x.o_ss = (unsigned)a.o_ss * 2, x.o_sh = (unsigned)a.o_sh * 2;
    x.k_sb = (unsigned)a.ks_sb * 2, x.k_ss = (unsigned)a.ks_ss * 2;
    const long long one = 0x7fffffffLL / 2, span = one / sb; // what block_offsets_fit grants one candidate, elements
    x.span = (int)(span < 1 << 20 ? span : 1 << 20); // (a window entry has 26 bits for it)
    x.div_n = make_fastdiv(sharers);
    x.div_run = make_fastdiv((unsigned)((a.S * a.G + 31) & -32));
    x.div_w = make_fastdiv(sharers * (unsigned)waves);
    return true;
}

// Positions of a window of align 1 at most.
inline long long packed_window(const Args &a)
{
    const long long tokens = 32 % a.G == 0 ? 32 / a.G : (a.G + 30) / a.G + 1;
    return a.S - 1 + tokens;
}

// Steps of a window, at most `most`; dense: lists of align 1 have no wider ones.
inline int packed_steps(const Args &a, int most, bool &dense)
{
    const long long window = packed_window(a);
    dense = window <= most * kTileKeys;
    return (int)((dense ? window : a.S) + kTileKeys - 1) / kTileKeys;
}

// Arithmetic of the lists, the same on the device and on the host (where tests run it).

struct Walk {
    int b, first, len; // candidate (global index), its first packed row, its length: wave-uniform
};

// Rows of a candidate of the given length in the list.
__host__ __device__ inline int packed_run(const Args &a, int len, int align) { return (len * a.G + align - 1) & -align; }

// Chooses the alignment, from the rows of either list.  Blocks across candidates are fewer, but their
// windows may go on to a second step: where a candidate's positions and a block's are more than 32, which with lengths of n
// is one block in n / (n + 32/G - 32).  A block takes the time of its tiles and some 6 more; a second step is counted
// as 18 - 1.4 for every prefix tile, what it costs and what blocks that memory bounds do not gain by being fewer.  us, across
// candidates and inside them, 1500 candidates, P 200 (500, P 250; 700, P 128): 32/32 heads: 20 positions: 222, 237 (81, 91; 107, 106);
// 17..25: 252, 246 (92, 94; 117, 114); 11..28: 246, 242 (87, 92; 119, 115); 22..32: 320, 300 (114, 103; 154, 143); 32/8: 28 positions: 217, 234 (83,
// 89; 96, 95); 32: 245, 243 (94, 93; 105, 105); 22..32: 217, 225 (84, 85; 93, 91); no second steps: 20: 153, 172 (57, 63; 65, 69).
// Where every wavefront has at most one block either way, blocks inside candidates: they take the shorter walk (32 candidates of 8..20,
// 32/8 heads, P 128: 11.6 us across, 11.1 inside).
template <int STEPS> __host__ __device__ inline int packed_align(const Args &a, bool dense, int tiles, int waves, int total, int total32)
{
    long long second = STEPS > 1 ? total - 32LL * (a.G - 1) * a.C : 0; // rows of blocks with a second step
    second = second > 0 ? second : 0;
    const int second_cost = tiles < 10 ? 180 - 14 * tiles : 40; // (tenths of a tile's time)
    const bool one = dense && total32 > 32 * waves && (long long)total * (10 * (tiles + 6)) + second_cost * second < (long long)total32 * (10 * (tiles + 6));
    return one ? 1 : kBlockRows;
}

__host__ __device__ inline int same_in_all_lanes(int x)
{
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_readfirstlane(x);
#else
    return x;
#endif
}

// Whether every run of the list is a full candidate's, so that a row's candidate is a division away.  No run is longer, so the sum says so.
// (Rows in all are not enough: with each candidate on blocks of its own, runs of 64, 32, 32 and 32 rows are as many as four candidates' 40.)
__host__ __device__ inline bool packed_even(const Args &a, int total, int align) { return total == a.C * packed_run(a, a.S, align); }

// The candidate (of one instruction's) of row r0 of such a list; its length is left to be filled in.  div_run: by a full candidate's run of whole blocks.
__host__ __device__ inline Walk walk_even(const Args &a, FastDiv div_run, int align, int r0)
{
    Walk w;
    w.b = same_in_all_lanes((int)(align == 1 ? fdiv(fdiv(r0, a.div_g), a.div_s) : fdiv(r0, div_run)));
    w.first = w.b * packed_run(a, a.S, align);
    w.len = 0;
    return w;
}

// The candidates of a block's rows.
struct BlockSpan {
    int b, first; // the first one, its first row in the list
    int last;     // the block's last row
    int width;    // positions of the window, one or more
    bool wide;    // it ends early: the next candidate is `span` or more away from the first one
};

// What window position l holds after the walk has entered the n-th candidate: (candidate - the first one) << 6 | position.
__host__ __device__ inline unsigned enter_window(unsigned entry, int l, int n, int at) { return l >= at ? (unsigned)(n << 6 | (l - at)) : entry; }

// Walks over the block of rows r0.. of a list of `total` rows: w, at or before the candidate of row r0, is left at the last row's or
// (wide) at the last one before the next, which may be empty.  len_of(b): length of candidate b; enter(n, at): the walk enters the
// n-th candidate after the first one, whose first position is the window's at-th.  It ends at the last candidate (cand_end is one
// past it), whatever the lengths say.
template <typename L, typename E>
__host__ __device__ __attribute__((always_inline)) inline BlockSpan walk_block(const Args &a, Walk &w, int r0, int total, int align, int span, int cand_end, L len_of,
                                                                               E enter)
{
    BlockSpan x;
    x.last = total - r0 < kBlockRows ? total - 1 : r0 + kBlockRows - 1;
    int end = w.first + packed_run(a, w.len, align);
    while (end <= r0 && w.b + 1 < cand_end) {
        w.first = end;
        ++w.b;
        w.len = len_of(w.b);
        end += packed_run(a, w.len, align);
    }
    x.b = w.b;
    x.first = w.first;
    x.wide = false;
    int at = 0; // window position of the walk's candidate's first
    while (end <= x.last && w.b + 1 < cand_end) {
        if (w.b + 1 - x.b >= span) {
            x.last = end - 1;
            x.wide = true;
            break;
        }
        at += w.len;
        w.first = end;
        ++w.b;
        w.len = len_of(w.b);
        end += packed_run(a, w.len, align);
        enter(w.b - x.b, at);
    }
    // The walk's candidate's positions: up to the last row's, none of an empty one.
    const int upto = x.last < w.first ? 0 : same_in_all_lanes((int)fdiv(x.last - w.first, a.div_g)) + 1;
    x.width = at + (upto < w.len ? upto : w.len);
    x.width = x.width > 1 ? x.width : 1;
    return x;
}

namespace {

typedef __attribute__((address_space(3))) int lds_int;

// Length of candidate b, b the same for the whole wavefront (as len_uniform; there are lengths).
__device__ inline int packed_len(const Args &a, int b)
{
    typedef const __attribute__((address_space(4))) int *const_int_ptr;
    return clamp_len(a, ((const_int_ptr)(unsigned long long)a.len)[__builtin_amdgcn_readfirstlane(b)]);
}

// Sum over the lanes up to and with this one.
__device__ inline int wave_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false); // row_shr:1, 2, 4, 8 ...
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false); // ... row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// The list of one instruction's packed rows, for a workgroup of 512 threads: the candidates in 256 chunks, one per thread
// of the first four wavefronts (the others request the prefix meanwhile).
constexpr int kLenWaves = 4, kLenChunks = kLenWaves * 64, kLenPerLane = kLenChunks / 64;
constexpr int kLenRound = 8;        // lengths per chunk that a thread fetches, and LDS holds, at a time
constexpr int kListInts = kLenChunks * (kLenRound + 2) + 2 * kLenWaves; // LDS words, in use from count_lengths to find_row
static_assert(kListInts * 4 <= kNW * kScrBytes, "the list's tables stand in the scratch tiles");

struct PackedList {
    int total, align; // rows
    bool even, full;  // every run is a full candidate's; nothing is padded
    int per_chunk;
    lds_int *lens;    // first, second, ... lengths of the chunks (of the last round), then rows of a wavefront's chunks up to and with each, for align 1 and for 32, and the wavefronts' rows
};

// Lengths k0 .. k0 + n - 1 (n <= kLenRound) of this thread's chunk.
__device__ inline void load_lengths(const Args &a, int cand0, int per_chunk, int k0, int n, int tid, int (&len)[kLenRound])
{
    const int lo = tid * per_chunk + k0;
#pragma unroll
    for (int k = 0; k < kLenRound; ++k) {
        len[k] = 0;
        if (k < n)
            len[k] = a.len[cand0 + (lo + k < a.C ? lo + k : a.C - 1)];
    }
}

// This thread's part: its chunk's rows for align 1 and 32.
struct ChunkRows {
    int rows, rows32;
};
__device__ inline void count_lengths(const Args &a, int per_chunk, int k0, int n, const int (&len)[kLenRound], lds_int *lens, int tid, ChunkRows &c)
{
#pragma unroll
    for (int k = 0; k < kLenRound; ++k)
        if (k < n) {
            const int l = tid * per_chunk + k0 + k < a.C ? clamp_len(a, len[k]) : 0;
            lens[k * kLenChunks + tid] = l;
            c.rows += l * a.G;
            c.rows32 += packed_run(a, l, kBlockRows);
        }
}

// Adds the chunks up (the first four wavefronts; a workgroup barrier follows).
__device__ inline void add_up(const ChunkRows &c, lds_int *lens, int tid)
{
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    lds_int *const tables = lens + kLenRound * kLenChunks, *const sums = tables + 2 * kLenChunks;
    const int upto = wave_scan(c.rows), upto32 = wave_scan(c.rows32);
    tables[tid] = upto;
    tables[kLenChunks + tid] = upto32;
    if ((tid & 63) == 63) {
        sums[wave] = upto;
        sums[kLenWaves + wave] = upto32;
    }
}

// The list of the alignment that is chosen (see packed_align).
template <int STEPS>
__device__ inline PackedList choose_list(const Args &a, const PackedArgs &pa, int tiles, int waves, int per_chunk, lds_int *lens)
{
    lds_int *const sums = lens + (kLenRound + 2) * kLenChunks;
    int total = 0, total32 = 0;
#pragma unroll
    for (int i = 0; i < kLenWaves; ++i) {
        total += sums[i];
        total32 += sums[kLenWaves + i];
    }
    total = __builtin_amdgcn_readfirstlane(total);
    total32 = __builtin_amdgcn_readfirstlane(total32);
    PackedList x;
    x.align = packed_align<STEPS>(a, pa.dense, tiles, waves, total, total32);
    x.total = x.align == 1 ? total : total32;
    x.even = packed_even(a, x.total, x.align);
    x.full = total == a.C * a.S * a.G;
    x.per_chunk = per_chunk;
    x.lens = lens;
    return x;
}

// Lane j: rows of the first (j + 1)/64 of the candidates (kLenPerLane chunks each).
__device__ inline int rows_upto(const PackedList &x, int lane)
{
    lds_int *const tables = x.lens + kLenRound * kLenChunks, *const before = x.align == 1 ? tables : tables + kLenChunks;
    lds_int *const sums = tables + 2 * kLenChunks + (x.align == 1 ? 0 : kLenWaves);
    int upto = before[kLenPerLane * lane + kLenPerLane - 1];
#pragma unroll
    for (int i = 0; i < kLenWaves - 1; ++i)
        upto += i < lane / (64 / kLenWaves) ? sums[i] : 0;
    return upto;
}

// The candidate of packed row r0 (one that exists).
__device__ inline Walk find_row(const Args &a, const PackedList &x, int cand0, int r0, int lane)
{
    lds_int *const tables = x.lens + kLenRound * kLenChunks, *const before = x.align == 1 ? tables : tables + kLenChunks;
    constexpr int n = kLenPerLane;
    const int upto = rows_upto(x, lane);
    const int g = __builtin_popcountll(__builtin_amdgcn_ballot_w64(upto <= r0)); // (below 64: the row exists)
    const int base = g > 0 ? __builtin_amdgcn_readlane(upto, g > 0 ? g - 1 : 0) : 0;
    const int part = before[n * g + (lane & (n - 1))] + (g % (64 / kLenWaves) ? base - before[g > 0 ? n * g - 1 : 0] : base);
    const int c = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < n && part <= r0));
    Walk w;
    w.b = __builtin_amdgcn_readfirstlane(cand0 + (n * g + c) * x.per_chunk);
    w.first = c > 0 ? __builtin_amdgcn_readlane(part, c > 0 ? c - 1 : 0) : base;
    const int chunk = n * g + c;
    w.len = x.per_chunk <= kLenRound ? __builtin_amdgcn_readfirstlane(x.lens[chunk]) : packed_len(a, w.b);
    return w;
}

// One block of 32 packed rows whose window takes up to STEPS steps of 32 positions.
template <int STEPS> struct PackedBlock {
    int r0, rows;   // its first row, its rows
    int b, first;   // the window's first candidate and that one's first packed row
    int width;      // the window's positions
    unsigned win;   // lane l (STEPS > 1; else lanes l and l + 32): window position l (the last one past the end): (candidate - b) << 6 | position
    unsigned win2;  // (STEPS == 3) lanes l and l + 32: position 64 + l
    unsigned o_off; // byte offset of the lane's row from the first candidate's first out row; bit 0: stored as zero
    unsigned sees;  // the window's keys that the lane's row sees: as bits, or (STEPS > 1) their last one and 256 times their first
    bool wide;      // its rows end early: the next candidate lies too far away for 32-bit offsets from the first one's rows
};

// The entry of window position pos.
template <int STEPS> __device__ inline unsigned window_entry(const PackedBlock<STEPS> &x, int pos)
{
    const unsigned e = (unsigned)__shfl((int)x.win, pos & 63, 64);
    if constexpr (STEPS == 3) {
        const unsigned e2 = (unsigned)__shfl((int)x.win2, pos & 31, 64);
        return pos < 64 ? e : e2;
    }
    return e;
}

// One lane's row of a packed block.  A row past its candidate's length (align 32) takes the query row and the keys of
// the last position that the block sees and is stored as zero; rows past the list's or the candidate's end are the last one once more.
struct PackedRow {
    int pos, gq;        // window position of its key, query head within the group
    unsigned from, own; // entries (as in `win`) of the row it loads and of the row it stores
};

template <int STEPS> __device__ inline PackedRow packed_row(const Args &a, const PackedBlock<STEPS> &x, int row, int align)
{
    PackedRow y;
    const int most = align > 1 ? a.S * a.G - 1 : x.r0 - x.first + x.rows - 1;
    int j = x.r0 - x.first + row;
    j = j < most ? j : most;
    const int pos = (int)fdiv(j, a.div_g);
    y.gq = j - pos * a.G;
    y.pos = pos < x.width ? pos : x.width - 1;
    y.from = window_entry(x, y.pos);
    y.own = pos < x.width ? y.from : (unsigned)(pos < a.S ? pos : a.S - 1);
    return y;
}

// Byte offset of an entry's row from that of the block's first candidate's first one.
__device__ inline unsigned packed_off(unsigned entry, unsigned sb, unsigned ss) { return __umul24(entry >> 6, sb) + __umul24(entry & 63, ss); }

// The block of packed rows r0..; w at or before the candidate of row r0, and left at its last row's.  q_off: byte offset of the
// lane's query row from the first candidate's first one; y: the lane's row.  Where candidates lie too far apart the block ends before
// the first such one (`wide`).
// len_of(b): length of candidate b.
template <int STEPS, typename F>
__device__ __attribute__((always_inline)) PackedBlock<STEPS> packed_block(const Args &a, const PackedArgs &pa, const Ctx &X, Walk &w, int r0, const PackedList &list,
                                                                          unsigned &q_off, PackedRow &y, F len_of)
{
    PackedBlock<STEPS> x;
    const int l = STEPS > 1 ? X.lane : X.c32;
    unsigned entry = l, entry2 = 64 + X.c32; // as if all were the first candidate's
    const BlockSpan sp = walk_block(a, w, r0, list.total, list.align, pa.span, X.cand0 + a.C, len_of, [&](int n, int at) __attribute__((always_inline)) {
        entry = enter_window(entry, l, n, at);
        if (STEPS == 3)
            entry2 = enter_window(entry2, 64 + X.c32, n, at);
    });
    x.r0 = r0;
    x.rows = sp.last - r0 + 1;
    x.b = sp.b;
    x.first = sp.first;
    x.width = sp.width;
    x.wide = sp.wide;
    const unsigned end1 = (unsigned)__builtin_amdgcn_readlane((int)entry, (sp.width - 1) & 63); // the last position's, whatever the walk ended at
    const unsigned end_entry = STEPS == 3 && sp.width > 64 ? (unsigned)__builtin_amdgcn_readlane((int)entry2, (sp.width - 65) & 63) : end1;
    x.win = l < x.width ? entry : end_entry;
    x.win2 = STEPS == 3 && 64 + X.c32 < x.width ? entry2 : end_entry;
    y = packed_row(a, x, X.c32, list.align);
    const unsigned rh = (unsigned)(X.head * a.G + y.gq);
    q_off = packed_off(y.from, pa.q_sb, pa.q_ss) + __umul24(rh, pa.q_sh);
    x.o_off = (packed_off(y.own, pa.o_sb, pa.o_ss) + __umul24(rh, pa.o_sh)) | (y.own == y.from ? 0u : 1u);
    const int lo = y.pos - (int)(y.from & 63); // the window's keys from its candidate's first to its own
    x.sees = STEPS > 1 ? (unsigned)(y.pos | lo << 8) : (2u << y.pos) - (1u << lo);
    return x;
}

template <int STEPS>
__device__ inline PackedBlock<STEPS> packed_block(const Args &a, const PackedArgs &pa, const Ctx &X, Walk &w, int r0, const PackedList &list, unsigned &q_off,
                                                PackedRow &y)
{
    return packed_block<STEPS>(a, pa, X, w, r0, list, q_off, y, [&](int b) { return packed_len(a, b); });
}

// The bits of the keys that the lane's row sees of window positions k0 .. k0 + 31, element e's at 8*(e/4) + e%4.
template <int STEPS> __device__ inline int sees_bits(const PackedBlock<STEPS> &x, int k0, int h)
{
    unsigned bits = x.sees;
    if constexpr (STEPS > 1) {
        const int end = (int)(x.sees & 255) + 1 - k0, lo = (int)(x.sees >> 8) - k0; // one past the last key, the first one
        bits = (end >= 32 ? ~0u : end > 0 ? (1u << end) - 1u : 0u) & (lo <= 0 ? ~0u : lo < 32 ? ~0u << lo : 0u);
    }
    return (int)(bits >> (4 * h));
}

// Q fragments of the block (layout as in load_q).
__device__ inline void load_q_packed(const Args &a, const PackedArgs &pa, const Ctx &X, int b, unsigned q_off, uintx4 (&dst)[8])
{
    const unsigned char *qrow = reinterpret_cast<const unsigned char *>(a.q) + (unsigned long long)(unsigned)b * pa.q_sb + (q_off + 16u * X.h);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
        dst[ks] = *reinterpret_cast<const uintx4 *>(qrow + 32 * ks);
}

// K fragments and V rows of the window's positions k0..k0+31 (layouts as in load_suffix_k and load_suffix_v; past the
// window its last position, which no row takes for that one's).
template <int STEPS> __device__ inline void load_window_k(const PackedArgs &pa, const Ctx &X, const PackedBlock<STEPS> &x, int k0, uintx4 (&kf)[8])
{
    const unsigned e = STEPS > 1 ? window_entry(x, k0 + X.c32) : x.win;
    const unsigned char *kp = reinterpret_cast<const unsigned char *>(X.ksg) + (unsigned long long)(unsigned)x.b * pa.k_sb +
                              (packed_off(e, pa.k_sb, pa.k_ss) + 16u * X.h);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
        kf[ks] = *reinterpret_cast<const uintx4 *>(kp + 32 * ks);
}

template <int STEPS> __device__ inline void load_window_v(const PackedArgs &pa, const Ctx &X, const PackedBlock<STEPS> &x, int k0, uintx4 (&vf)[2][4])
{
    const unsigned char *base = reinterpret_cast<const unsigned char *>(X.vsg) + (unsigned long long)(unsigned)x.b * pa.k_sb;
#pragma unroll
    for (int j = 0; j < 2; ++j) { // (fragment (dt, u) = (it, h) of load_suffix_v)
        const unsigned e = window_entry(x, k0 + 16 * j + 8 * X.h + X.sv_row_lo);
        const unsigned char *vp = base + (packed_off(e, pa.k_sb, pa.k_ss) + (unsigned)X.sv_chunk_lo * 16u);
#pragma unroll
        for (int it = 0; it < 4; ++it)
            vf[j][it] = *reinterpret_cast<const uintx4 *>(vp + 64 * it);
    }
}

// Normalise and store the block (as store_block).
template <int STEPS>
__device__ inline void store_packed(const Args &a, const PackedArgs &pa, const Ctx &X, const PackedBlock<STEPS> &x, int align, float m, float l, const floatx16 (&o)[4])
{
    const float ltot = sum_of_halves(l);
    const float inv = 1.0f / ltot;
    const bool rvalid = !(x.o_off & 1);
    unsigned char *base = reinterpret_cast<unsigned char *>(a.out) + (unsigned long long)(unsigned)x.b * pa.o_sb;
    unsigned short *dst[4];
    bool dst_ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const unsigned off = (unsigned)__shfl((int)x.o_off, 8 * u + (X.lane >> 3), 64) & ~1u;
        dst[u] = reinterpret_cast<unsigned short *>(base + (off + 16u * (X.lane & 7)));
        // (lanes past the last row are that row once more, with its bits: stored too, so that the number of stores in flight is
        // known and the wait for the next block's Q, requested before them, is not one for the stores)
        dst_ok[u] = true;
    }
    store_rows(X, dst, dst_ok, rvalid, inv, o);
    if (a.lse) {
        const PackedRow y = packed_row(a, x, X.c32, align); // (takes entries from all lanes)
        if (X.h == 0)
            a.lse[((long long)(x.b + (int)(y.own >> 6)) * a.Hq + X.head * a.G + y.gq) * a.S + (int)(y.own & 63)] =
                rvalid ? (m + __builtin_log2f(ltot)) * kLn2 : -INFINITY;
    }
}

// A window step after the first: raw scores s of 32 positions of which the row sees those whose bits are set (shifted for
// the lane's half), weights relative to the fixed reference m, value product through the scratch tile.
__device__ inline void window_step_fixed(const Ctx &X, int bits, const floatx16 &s, float m, float &l, const uintx4 (&svf)[2][4], floatx16 (&o)[4])
{
    unsigned pk[8];
    float rs = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
        const float p0 = keep_if_bit(fast_exp2(__builtin_fmaf(s[e], X.c, -m)), bits, 8 * (e >> 2) + (e & 3));
        const float p1 = keep_if_bit(fast_exp2(__builtin_fmaf(s[e + 1], X.c, -m)), bits, 8 * ((e + 1) >> 2) + ((e + 1) & 3));
        rs += p0;
        rs += p1;
        pk[e >> 1] = pack_bf16(p0, p1);
    }
    l += rs;
    pv_from_scratch(X, svf[0], as_bf16x8(uintx4{pk[0], pk[1], pk[2], pk[3]}), o);
    pv_from_scratch(X, svf[1], as_bf16x8(uintx4{pk[4], pk[5], pk[6], pk[7]}), o);
}

// Zeros for candidate b's (of the given length) rows past those that its blocks store, of this KV head's query heads (whole rows, 16 lanes each), in a
// tensor with the given strides (bytes), and minus infinity in lse (null: none).
__device__ inline void store_padding(const Args &a, const Ctx &X, int b, int len, int align, void *out, unsigned sb, unsigned ss, unsigned sh, float *lse)
{
    const int all = a.S * a.G, from = packed_run(a, len, align);
    unsigned char *base = reinterpret_cast<unsigned char *>(out) + (unsigned long long)(unsigned)b * sb + (unsigned)(X.head * a.G) * sh;
    for (int r = from + (X.lane >> 4); r < all; r += 4) {
        const unsigned t = fdiv(r, a.div_g), gq = r - t * a.G;
        __builtin_nontemporal_store(uintx4{0, 0, 0, 0}, reinterpret_cast<uintx4 *>(base + (__umul24(t, ss) + __umul24(gq, sh) + 16u * (X.lane & 15))));
    }
    if (lse)
        for (int r = from + X.lane; r < all; r += 64) {
            const unsigned t = fdiv(r, a.div_g), gq = r - t * a.G;
            lse[((long long)b * a.Hq + X.head * a.G + (int)gq) * a.S + (int)t] = -INFINITY;
        }
}

// The classic online softmax over a packed block whatever its rows and its prefix are: the block's rows and Q (w as in walk_block, and left
// for the next block), and, after the prefix, its window and the store.
template <int STEPS> struct GeneralBlock {
    PackedBlock<STEPS> x;
    PackedRow y;
    Row row;
    RowState st;
    uintx4 q[8];
};

template <int STEPS>
__device__ __attribute__((always_inline)) void packed_general_begin(const Args &a, const PackedArgs &pa, const Ctx &X, Walk &w, int r0, const PackedList &list,
                                                                    GeneralBlock<STEPS> &g)
{
    unsigned q_off;
    PackedArgs far = pa;
    far.span = 1 << 26; // (the offsets that do not reach are not used here)
    g.x = packed_block<STEPS>(a, far, X, w, r0, list, q_off, g.y);
    g.row.rb = g.x.b + (g.y.from >> 6);
    g.row.ri = g.y.from & 63;
    g.row.rh = X.head * a.G + g.y.gq;
    load_q(a, X, g.row, g.q);
    g.st.m = -INFINITY;
    g.st.l = 0.f;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            g.st.o[dt][e] = 0.f;
}

template <int STEPS> __device__ __attribute__((always_inline)) void packed_general_end(const Args &a, const Ctx &X, GeneralBlock<STEPS> &g)
{
    for (int k0 = 0; k0 < g.x.width; k0 += kTileKeys) {
        uintx4 kf[8], vf[2][4];
        auto row_of = [&](const unsigned short *base, int pos) {
            const unsigned e = window_entry(g.x, pos);
            return base + (long long)(g.x.b + (int)(e >> 6)) * a.ks_sb + (long long)(e & 63) * a.ks_ss;
        };
        const unsigned short *kp = row_of(X.ksg, k0 + X.c32) + 8 * X.h;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            kf[ks] = ld_global16(kp + 16 * ks);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const unsigned short *vp = row_of(X.vsg, k0 + 16 * j + 8 * X.h + X.sv_row_lo) + 8 * X.sv_chunk_lo;
#pragma unroll
            for (int it = 0; it < 4; ++it)
                vf[j][it] = ld_global16(vp + 32 * it);
        }
        const unsigned bits = (unsigned)sees_bits(g.x, k0, X.h);
        floatx16 s;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            s[e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks]), as_bf16x8(g.q[ks]), s, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 16; ++e)
            s[e] = bits >> (8 * (e >> 2) + (e & 3)) & 1 ? s[e] : -INFINITY;
        bf16x8 pf[2];
        softmax_tile(s, g.st, X.c, pf);
        pv_from_scratch(X, vf[0], pf[0], g.st.o);
        pv_from_scratch(X, vf[1], pf[1], g.st.o);
    }
    const float ltot = sum_of_halves(g.st.l);
    unsigned short *dst[4];
    bool dst_ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) { // (entries and heads of the rows that this lane stores come from the lanes that own them)
        const int from = 8 * u + (X.lane >> 3);
        const unsigned e = (unsigned)__shfl((int)g.y.own, from, 64);
        const int rh = __shfl(g.row.rh, from, 64);
        dst[u] = reinterpret_cast<unsigned short *>(a.out) + (long long)(g.x.b + (int)(e >> 6)) * a.o_sb + (long long)(e & 63) * a.o_ss + (long long)rh * a.o_sh +
                 8 * (X.lane & 7);
        dst_ok[u] = true;
    }
    store_rows(X, dst, dst_ok, g.y.own == g.y.from, 1.0f / ltot, g.st.o);
    if (a.lse && X.h == 0)
        a.lse[((long long)(g.x.b + (int)(g.y.own >> 6)) * a.Hq + g.row.rh) * a.S + (int)(g.y.own & 63)] =
            g.y.own == g.y.from ? (g.st.m + __builtin_log2f(ltot)) * kLn2 : -INFINITY;
}

} // namespace
} // namespace pskv
