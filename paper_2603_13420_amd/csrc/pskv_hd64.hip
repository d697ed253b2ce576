// Matrix-core kernels for bf16 tensors with heads of 64 columns: forward pass and the gradients of
// the suffix side, any prefix length, suffix shape and query-head group.
//
// Layouts and formulation are those of pskv_mfma.hpp (32-row blocks of the stacked rows
// r = (b*S + i)*G + g, 32-key tiles, a lane owns a query column), with two differences.
//   - Weights, and score gradients, enter the second products as THREE bf16 numbers that add up to the
//     fp32 number to the last bit (8 of its 24 significant bits each, cut off and not rounded), as the vector
//     kernels that serve the other head dimensions have them in fp32.  Half the columns leave the matrix
//     cores with time to spare: two further products cost less than the precision is worth (7 to 16 % of a call
//     over two parts, which hold 16 bits).
//   - The own suffix keys of all candidates a block of rows touches form ONE list, cut into 32-key
//     steps: a row sees a contiguous run of it, and a block that straddles short candidates takes one
//     or two steps where one step (or more) per candidate would be mostly empty.
//
// At these sizes (heads of half the width belong to small models) much is latency: a
// persistent workgroup of 8 wavefronts, two per compute unit, copies as much of its head's prefix
// into LDS as fits, and its wavefronts walk over the row blocks independently.  Longer prefixes go
// through the same LDS in chunks.
//
// 256 candidates of 5 to 33 rows, 177 prefix rows, 14/2 heads: 300 us in the vector kernel, 20.9 us here (22.6 us with the
// prefix copied through registers, 32 bytes of a row at a time, and transposed in LDS, and the first tile tried as a later
// one before its maximum was taken).
#include "pskv_mfma.hpp"
#include <type_traits>

namespace pskv {
namespace {

constexpr int kW = 64;                    // head dimension
constexpr int kKS = kW / 16;              // contraction steps of the first products
constexpr int kDT = kW / 32;              // column tiles of the second ones
constexpr int kImg = kTileKeys * kW * 2;  // an image of a 32-key tile: 4 KB
constexpr int kFwdWaves = 8;

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ inline floatx16 zero16()
{
    floatx16 z;
#pragma unroll
    for (int e = 0; e < 16; ++e)
        z[e] = 0.f;
    return z;
}
__device__ inline floatx16 mma(bf16x8 a, bf16x8 b, floatx16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ inline bf16x8 lds_frag(lds_u8 *p) { return as_bf16x8(*(lds_u128 *)p); }

// Fragments (contraction steps 0 and 1) of 16 values in three parts: p[0] + p[1] + p[2] is the value, exactly.
// (An infinity leaves NaN in the later parts: see to_form_anew.)
constexpr int kParts = 3;
struct Split {
    bf16x8 p[kParts][2];
};
__device__ inline Split split16(float (&v)[16])
{
    Split s;
#pragma unroll
    for (int part = 0; part < kParts; ++part) {
        unsigned w[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            // the upper halves of two numbers
            w[i] = __builtin_amdgcn_perm(__float_as_uint(v[2 * i + 1]), __float_as_uint(v[2 * i]), 0x07060302);
            if (part + 1 < kParts) {
                v[2 * i] -= __uint_as_float(w[i] << 16);
                v[2 * i + 1] -= __uint_as_float(w[i] & 0xffff0000u);
            }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
            s.p[part][j] = as_bf16x8(uintx4{w[4 * j], w[4 * j + 1], w[4 * j + 2], w[4 * j + 3]});
    }
    return s;
}

// Fragment (column tile dt, contraction step j) of a transposed operand
// from a "transposable" image (the V image of pskv_mfma.hpp), through the transposing read.
__device__ inline bf16x8 frag_tr(lds_u8 *img, int dt, int j, int lane)
{
    short4v lo = lds_read_tr(img + ((dt * 2 + j) * 2 + 0) * 512 + lane * 8), hi = lds_read_tr(img + ((dt * 2 + j) * 2 + 1) * 512 + lane * 8);
    short8v v8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    bf16x8 f;
    __builtin_memcpy(&f, &v8, 16);
    return f;
}
// Which 16-byte chunk (key, column chunk) belongs at chunk position p (0..255) of a transposable image.
__device__ inline void transposable_slot(int p, int &key, int &chunk)
{
    const int f = p >> 5, q = p & 31; // fragment (dt, j, u), slot pair within it
    key = 16 * ((f >> 1) & 1) + 8 * (f & 1) + 4 * (q >> 4) + ((q & 7) >> 1);
    chunk = 4 * (f >> 2) + 2 * ((q >> 3) & 1) + (q & 1);
}

// The rows of one 32-row block, as the lane of row c32 sees them.
struct Rows {
    int b, i, h, len;        // candidate, suffix position, query head, clamped suffix length
    bool exists, valid;
    int bl0, bl1, tok0, tok1; // candidates within the instruction and tokens that the block covers
};

// The list of own keys: keys 0 .. n_c - 1 of every candidate c of the block, in order; n_c is one more
// than the last key that any of the block's rows sees.  visit(candidate, first slot, n_c).
template <typename F> __device__ inline int own_keys(const Args &a, const Ctx &X, const Rows &x, F visit)
{
    int n = 0;
    for (int bl = x.bl0; bl <= x.bl1; ++bl) {
        const int b = X.cand0 + bl, len = len_uniform(a, b);
        const int lo = x.tok0 - bl * a.S > 0 ? x.tok0 - bl * a.S : 0;
        const int hi = x.tok1 - bl * a.S < len - 1 ? x.tok1 - bl * a.S : len - 1;
        const int nc = lo < len ? hi + 1 : 0;
        visit(b, n, nc);
        n += nc;
    }
    return n;
}
__device__ inline Rows make_rows(const Args &a, const Ctx &X, int blk)
{
    Rows x;
    const int r0 = blk * kBlockRows, last = r0 + kBlockRows - 1 < X.Mtot ? r0 + kBlockRows - 1 : X.Mtot - 1;
    const int r = r0 + X.c32 < X.Mtot ? r0 + X.c32 : X.Mtot - 1;
    x.exists = r0 + X.c32 < X.Mtot;
    const int tok = (int)fdiv(r, a.div_g), bl = (int)fdiv(tok, a.div_s);
    x.b = X.cand0 + bl;
    x.i = tok - bl * a.S;
    x.h = X.head * a.G + (r - tok * a.G);
    // (By a vector load: the walk over the block's candidates that finds the lengths as scalars would stand before every
    // address of the row's.  us, 14/2 heads unless stated, from such a walk and so: 501 candidates x 45..87 positions, P 35: 81.4,
    // 76.7; 313 x 75, P 43: 45.2, 43.1; 205 x 86..110, P 34, 32/8: 115.6, 112.6.)
    x.len = a.len ? clamp_len(a, a.len[x.b]) : a.S;
    x.valid = x.exists && x.i < x.len;
    x.tok0 = (int)fdiv(r0, a.div_g);
    x.tok1 = (int)fdiv(last, a.div_g);
    x.bl0 = (int)fdiv(x.tok0, a.div_s);
    x.bl1 = (int)fdiv(x.tok1, a.div_s);
    return x;
}
// The slots of the block's list, and where those of the lane's row begin.
struct OwnList {
    int n, first;
};
__device__ inline OwnList own_list(const Args &a, const Ctx &X, const Rows &x)
{
    OwnList l;
    l.first = 0;
    l.n = own_keys(a, X, x, [&](int b, int first, int) { l.first = b == x.b ? first : l.first; });
    return l;
}

// Element offset (from the suffix tensors of this head) of the row in slot k0 + c32 of the list, the last
// slot standing in for those behind it.  (The list holds at least one.)
__device__ inline long long own_row(const Args &a, const Ctx &X, const Rows &x, int k0)
{
    const int slot = k0 + X.c32;
    long long off = 0;
    own_keys(a, X, x, [&](int b, int first, int nc) {
        if (nc > 0 && slot >= first)
            off = (long long)b * a.ks_sb + (long long)(slot - first < nc ? slot - first : nc - 1) * a.ks_ss;
    });
    return off;
}
__device__ inline void load_row(const void *base, long long off, int h, uintx4 (&f)[kKS])
{
    const unsigned short *p = reinterpret_cast<const unsigned short *>(base) + off + 8 * h;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks)
        f[ks] = ld_global16(p + 16 * ks);
}

// 32 own rows of the list (slots from k0; `row`: this lane's own, from own_row) in transposable order into
// the wavefront's scratch image.
__device__ inline void own_to_scratch(const Ctx &X, const unsigned short *base, long long row)
{
    uintx4 v[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        int key, chunk;
        transposable_slot(it * 64 + X.lane, key, chunk);
        v[it] = ld_global16(base + shfl64(row, key) + chunk * 8);
    }
#pragma unroll
    for (int it = 0; it < 4; ++it)
        *(lds_u128 *)(X.scr + it * 1024 + X.lane * 16) = v[it];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Rows of the block held as row-major fragments (lane (row c32, half h): columns 16*ks + 8*h ..+7) into a
// transposable image.
__device__ inline void rows_to_image(const Ctx &X, lds_u8 *img, const uintx4 (&f)[kKS])
{
    lds_u8 *dst = img + (((X.c32 >> 4) * 2) + ((X.c32 >> 3) & 1)) * 512 + (16 * ((X.c32 >> 2) & 1) + 2 * (X.c32 & 3) + X.h) * 16;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks)
        *(lds_u128 *)(dst + (ks >> 1) * 2048 + (ks & 1) * 128) = f[ks];
}

// Stores a block held as transposed accumulators (lane column = row): o[dt][4kk + t] is column
// 32dt + 8kk + 4h + t.  The two lanes of a row trade half of their pieces, so that each holds runs of 8
// columns: 32 contiguous bytes of a row per instruction.
__device__ inline void store_transposed(unsigned short *row, int h, bool exists, bool valid, float scale, const floatx16 (&o)[kDT])
{
    const float f = valid ? scale : 0.f;
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
            unsigned w[4]; // columns 0,1 and 2,3 of piece kk = 2pr, then of piece 2pr + 1
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = 8 * pr + 2 * i;
                w[i] = pack_bf16(mul_zero_wins(o[dt][e], f), mul_zero_wins(o[dt][e + 1], f));
            }
            // the upper half-wave's piece 2pr against the lower one's piece 2pr + 1
            const auto x = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
            const auto y = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
            if (exists)
                __builtin_nontemporal_store(uintx4{x[0], y[0], x[1], y[1]}, reinterpret_cast<uintx4 *>(row + 32 * dt + 16 * pr + 8 * h));
        }
}

// ------------------------------------------------------------------------------------------
// The products take hidden terms - keys of the block's other candidates, keys behind the row's position,
// rows that do not see the key - with a weight of zero, and zero times an infinity or NaN among them is NaN.
// That is all such a term can do (hidden scores are replaced before anything is made of them).  So a wavefront
// whose valid sums hold a NaN goes over its blocks once more behind its loops (where this costs the loops
// no registers): every lane forms those columns of the rows it has stored anew, alone, from the terms that the row
// has, and stores them over the others.
// ------------------------------------------------------------------------------------------
__device__ inline float lane_dot(const unsigned short *x, const unsigned short *y)
{
    float acc = 0.f;
#pragma unroll 1
    for (int c = 0; c < kW; c += 8) {
        const uintx4 u = ld_global16(x + c), v = ld_global16(y + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc = __builtin_fmaf(__uint_as_float(u[e] << 16), __uint_as_float(v[e] << 16), acc);
            acc = __builtin_fmaf(__uint_as_float(u[e] & 0xffff0000u), __uint_as_float(v[e] & 0xffff0000u), acc);
        }
    }
    return acc;
}
// Eight columns of a sum over rows.
struct Columns {
    float v[8] = {};
    __device__ void add(float w, const unsigned short *row)
    {
        const uintx4 u = ld_global16(row);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[2 * e] = __builtin_fmaf(w, __uint_as_float(u[e] << 16), v[2 * e]);
            v[2 * e + 1] = __builtin_fmaf(w, __uint_as_float(u[e] & 0xffff0000u), v[2 * e + 1]);
        }
    }
    __device__ void store(unsigned short *row, float scale) const
    {
        uintx4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            y[e] = pack_bf16(v[2 * e] * scale, v[2 * e + 1] * scale);
        *reinterpret_cast<uintx4 *>(row) = y;
    }
};
// Whether eight stored columns are to be formed anew: a NaN is among them, or nothing but zeros (what a row without a
// finite score was stored as).
__device__ inline bool to_form_anew(const unsigned short *row)
{
    const uintx4 y = ld_global16(row);
    bool nan = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float lo = __uint_as_float(y[e] << 16), hi = __uint_as_float(y[e] & 0xffff0000u);
        nan |= lo != lo || hi != hi;
    }
    return nan || (y[0] | y[1] | y[2] | y[3]) == 0;
}
// Calls f(K row, V row) for the keys that the lane's row sees.
template <typename F> __device__ inline void for_visible_keys(const Args &a, const Ctx &X, const Rows &x, F f)
{
#pragma unroll 1
    for (int j = 0; j < X.P; ++j)
        f(X.kpg + (long long)j * a.kp_sp, X.vpg + (long long)j * a.kp_sp);
    const unsigned short *ks = X.ksg + (long long)x.b * a.ks_sb, *vs = X.vsg + (long long)x.b * a.ks_sb;
#pragma unroll 1
    for (int j = 0; j <= x.i; ++j)
        f(ks + (long long)j * a.ks_ss, vs + (long long)j * a.ks_ss);
}
__device__ inline bool has_nan(const floatx16 (&o)[kDT])
{
    bool nan = false;
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e)
            nan |= o[dt][e] != o[dt][e];
    return nan;
}

__device__ inline Ctx make_hd64_ctx(const Args &a, int tid)
{
    Ctx X;
    X.lane = tid & 63;
    X.h = X.lane >> 5;
    X.c32 = X.lane & 31;
    X.Mtot = a.C * a.S * a.G;
    X.c = a.scale * kLog2e;
    return X;
}

// Prefix rows of tiles t0 .. t0 + n - 1 into LDS (whole workgroup of 8 wavefronts), K and V of tile t as half images
// (pskv_mfma.hpp; at 64 columns an image is a whole tile) at img + (t - t0) * kTile.  The last row stands in for
// rows behind the prefix (never visible).
// All 1 KB pieces - 8 rows, whole cache lines - are requested straight into LDS at once: no registers, one round
// trip.  Between the request and the barrier that ends stage_finish there is room for other requests.
constexpr int kTile = 2 * kImg;
__device__ inline void stage_request(const Args &a, const Ctx &X, lds_u8 *img, int t0, int n, int tid)
{
    asm volatile("" : "+v"(tid)); // (worked out here: nothing held across the callers' loops)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int g = wave & 3; // this wavefront's pieces: rows 8g .. 8g+7 of a tile
    const unsigned short *src = wave & 4 ? X.vpg : X.kpg;
    const unsigned k = ((unsigned)lane >> 3) ^ (g & 1); // what half_put puts at lane*16
    const int row = 8 * g + (int)k, chunk = (int)(((unsigned)lane & 7) ^ half_swz(k)), last = X.P - 1; // (P > 0: there is a tile)
    __syncthreads(); // every wavefront is done with what was there
    for (int t = 0; t < n; ++t) {
        const int key = (t0 + t) * kTileKeys + row;
        request_to_lds(src + ((long long)(key < last ? key : last) * a.kp_sp + chunk * 8), img + t * kTile + wave * 1024);
    }
}
__device__ inline void stage_finish()
{
    PSKV_WAIT_VM(0);
    __syncthreads();
}

__device__ inline bf16x8 tile_row_frag(const TilePlaces &x, lds_u8 *img, int i) { return lds_frag(img + x.row[i]); }
__device__ inline bf16x8 tile_col_frag(const TilePlaces &x, lds_u8 *img, int d, int j)
{
    short4v lo = lds_read_tr(img + x.col[d][0] + j * 2048), hi = lds_read_tr(img + x.col[d][1] + j * 2048 + 1024);
    short8v v8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    bf16x8 f;
    __builtin_memcpy(&f, &v8, 16);
    return f;
}

// How a persistent grid is laid over the (instruction, KV head) pairs: see resident_general_kernel.
struct Spread {
    int per_vh, vh_slots, chunk; // workgroups per pair, pairs served at a time, tiles that fit into LDS
};
// The first of the blocks that this workgroup's wavefronts take in their round `it` (at or behind the number of blocks: none).
__device__ inline int round_base(const Spread &sp, int waves, int it) { return ((blockIdx.x / sp.vh_slots) + it * sp.per_vh) * waves; }

// f(arguments, context, row) for the valid rows of this wavefront's blocks in a walk of `waves` wavefronts per workgroup, for
// a path hardly ever taken.  (A kernel's first parameter is, or begins with, Args.)
template <typename F> __device__ inline void for_stored_rows(const Spread &sp, int waves, int tid, F f)
{
    const Args &a = first_parameter<Args>();
    asm volatile("" : "+v"(tid)); // (nothing of this is worked out ahead)
    Ctx X = make_hd64_ctx(a, tid);
    const int nblocks = (X.Mtot + kBlockRows - 1) / kBlockRows, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int vh = blockIdx.x % sp.vh_slots; vh < a.Np * a.Hkv; vh += sp.vh_slots) {
        set_vhead(a, X, vh);
        for (int it = 0, blk; (blk = round_base(sp, waves, it) + wave) < nblocks; ++it) {
            const Rows x = make_rows(a, X, blk);
            if (x.valid)
                f(a, X, x);
        }
    }
}

struct FwdState {
    float m, l;
    floatx16 o[kDT];
};

// O^T += V^T P^T (FRESH: O^T = V^T P^T); vf(dt, j) hands out the V^T fragments.
template <bool FRESH, typename VF> __device__ inline void add_products(float (&p)[16], FwdState &st, VF vf)
{
    const Split w = split16(p);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) {
            const bf16x8 v = vf(dt, j);
            if (FRESH && j == 0)
                st.o[dt] = zero16();
#pragma unroll
            for (int part = kParts - 1; part >= 0; --part) // (the small ones first)
                st.o[dt] = mma(v, w.p[part][j], st.o[dt]);
        }
}

// Softmax of a tile's raw scores (-inf: not visible) against the row's reference, rescaling only when a weight
// comes out huge (cf. softmax_tile), and the value product.
template <typename VF> __device__ inline void weigh_tile(const floatx16 &s, float c, FwdState &st, VF vf)
{
    float p[16], rs = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        p[e] = fast_exp2(__builtin_fmaf(s[e], c, -st.m));
        rs += p[e];
    }
    if (__builtin_amdgcn_ballot_w64(!(rs < kBig)) != 0) {
        float tmax = s[0];
#pragma unroll
        for (int e = 1; e < 16; ++e)
            tmax = fmaxf(tmax, s[e]);
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
        const float mnew = fmaxf(st.m, tmax * c);
        const float msafe = mnew == -INFINITY ? 0.f : mnew; // nothing visible yet: weights all 0
        const float alpha = fast_exp2(st.m - msafe);
        st.l *= alpha;
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt)
            st.o[dt] *= alpha;
        st.m = mnew;
        rs = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            p[e] = fast_exp2(__builtin_fmaf(s[e], c, -msafe));
            rs += p[e];
        }
    }
    st.l += rs;
    add_products<false>(p, st, vf);
}

// The same for a row's first tile.
template <typename VF> __device__ inline void weigh_first(const floatx16 &s, float c, FwdState &st, VF vf)
{
    float tmax = s[0];
#pragma unroll
    for (int e = 1; e < 16; ++e)
        tmax = fmaxf(tmax, s[e]);
    st.m = fmaxf(tmax, __shfl_xor(tmax, 32, 64)) * c;
    const float msafe = st.m == -INFINITY ? 0.f : st.m;
    float p[16];
    st.l = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        p[e] = fast_exp2(__builtin_fmaf(s[e], c, -msafe));
        st.l += p[e];
    }
    add_products<true>(p, st, vf);
}

__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(4)))
void hd64_fwd_kernel(Args a, Spread sp)
{
    extern __shared__ __align__(256) unsigned char smem_generic[];
    lds_u8 *img = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X = make_hd64_ctx(a, tid);
    X.scr = img + sp.chunk * kTile + wave * kImg;
    const TilePlaces tp = tile_places(half_places(X.lane));
    const int nblocks = (X.Mtot + kBlockRows - 1) / kBlockRows, VH = a.Np * a.Hkv;
    bool bad = false;

    for (int vh = blockIdx.x % sp.vh_slots; vh < VH; vh += sp.vh_slots) {
        set_vhead(a, X, vh);
        const int T = (X.P + kTileKeys - 1) / kTileKeys;
        const bool resident = T <= sp.chunk;
        if (resident) {
            stage_request(a, X, img, 0, T, tid);
            stage_finish();
        }
        // (The workgroup's wavefronts go through this loop together - barriers inside - unless the prefix is resident.)
        // Nothing is asked for while the prefix is on its way: the barrier would wait for that too.  us, the first
        // block's query rows requested there, and so: 428 candidates x 13 positions, P 64, 14/2 heads: 15.0, 12.7; 143 x 21, P 64, 32/8:
        // 15.7, 13.7; 256 x 5..33, P 177, 14/2: 20.9 both.
        for (int it = 0;;) { // (the launcher gives every workgroup a first round)
            const int blk = round_base(sp, kFwdWaves, it) + wave;
            const bool has = blk < nblocks;
            const Rows x = make_rows(a, X, has ? blk : nblocks - 1);
            const OwnList own = own_list(a, X, x); // (here and not behind the tiles: its loads pass beside those of the rows)
            const bool work = has && __builtin_amdgcn_ballot_w64(x.valid) != 0;
            uintx4 q[kKS];
            load_row(a.q, (long long)x.b * a.q_sb + (long long)(x.valid ? x.i : 0) * a.q_ss + (long long)x.h * a.q_sh, X.h, q);
            FwdState st;
            st.m = -INFINITY;
            st.l = 0.f;
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt)
                st.o[dt] = zero16();

            for (int t0 = 0; t0 < T; t0 += sp.chunk) {
                const int n = T - t0 < sp.chunk ? T - t0 : sp.chunk;
                if (!resident) {
                    stage_request(a, X, img, t0, n, tid);
                    stage_finish();
                }
                if (!work)
                    continue;
                auto tile = [&](int t, auto first) __attribute__((always_inline)) {
                    lds_u8 *ki = img + t * kTile, *vi = ki + kImg;
                    floatx16 s = zero16();
#pragma unroll
                    for (int ks = 0; ks < kKS; ++ks)
                        s = mma(tile_row_frag(tp, ki, ks), as_bf16x8(q[ks]), s);
                    int nv = X.P - (t0 + t) * kTileKeys - 4 * X.h; // element e holds key 8*(e/4) + e%4 + 4*h of the tile
                    asm volatile("" : "+v"(nv)); // (the first tile's comparisons stay here: ahead of the loops their 16 results would be spilled)
                    if ((t0 + t + 1) * kTileKeys > X.P)
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            if (8 * (e >> 2) + (e & 3) >= nv)
                                s[e] = -INFINITY;
                    auto v = [&](int dt, int j) { return tile_col_frag(tp, vi, dt, j); };
                    if constexpr (decltype(first)::value)
                        weigh_first(s, X.c, st, v);
                    else
                        weigh_tile(s, X.c, st, v);
                };
                int t = 0;
                if (t0 == 0)
                    tile(t++, std::true_type{});
                for (; t < n; ++t)
                    tile(t, std::false_type{});
            }
            if (work) {
                for (int k0 = 0; k0 < own.n; k0 += kTileKeys) {
                    const long long row = own_row(a, X, x, k0);
                    uintx4 kf[kKS];
                    load_row(X.ksg, row, X.h, kf);
                    own_to_scratch(X, X.vsg, row);
                    floatx16 s = zero16();
#pragma unroll
                    for (int ks = 0; ks < kKS; ++ks)
                        s = mma(as_bf16x8(kf[ks]), as_bf16x8(q[ks]), s);
                    const int rel = k0 + 4 * X.h - own.first; // the row sees slots first .. first + i
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        s[e] = (unsigned)(rel + 8 * (e >> 2) + (e & 3)) <= (unsigned)x.i ? s[e] : -INFINITY;
                    weigh_tile(s, X.c, st, [&](int dt, int j) { return frag_tr(X.scr, dt, j, X.lane); });
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
            }
            if (has) {
                const float l = st.l + __shfl_xor(st.l, 32, 64);
                store_transposed(reinterpret_cast<unsigned short *>(a.out) + (long long)x.b * a.o_sb + (long long)x.i * a.o_ss +
                                     (long long)x.h * a.o_sh,
                                 X.h, x.exists, x.valid, 1.0f / l, st.o);
                const float lse2 = l != 0.f ? st.m + __builtin_log2f(l) : NAN; // (no sum: every score is -inf, and the result NaN)
                if (a.lse && x.exists && X.h == 0)
                    a.lse[((long long)x.b * a.Hq + x.h) * a.S + x.i] = x.valid ? lse2 * kLn2 : -INFINITY;
                bad |= __builtin_amdgcn_ballot_w64(x.valid && (has_nan(st.o) || l == 0.f)) != 0;
            }
            if (round_base(sp, kFwdWaves, ++it) >= nblocks)
                break;
        }
    }
    if (bad) // (see to_form_anew)
        for_stored_rows(sp, kFwdWaves, tid, [](const Args &a, const Ctx &X, const Rows &x) {
            unsigned short *out = reinterpret_cast<unsigned short *>(a.out) + (long long)x.b * a.o_sb + (long long)x.i * a.o_ss + (long long)x.h * a.o_sh;
            const unsigned short *q = reinterpret_cast<const unsigned short *>(a.q) + (long long)x.b * a.q_sb + (long long)x.i * a.q_ss + (long long)x.h * a.q_sh;
#pragma unroll 1
            for (int c = 8 * X.h; c < kW; c += 16) {
                if (!to_form_anew(out + c))
                    continue;
                float m = -INFINITY, l = 0.f;
                for_visible_keys(a, X, x, [&](const unsigned short *k, const unsigned short *) { m = fmaxf(m, lane_dot(q, k) * X.c); });
                Columns y;
                for_visible_keys(a, X, x, [&](const unsigned short *k, const unsigned short *v) {
                    const float p = fast_exp2(__builtin_fmaf(lane_dot(q, k), X.c, -m));
                    l += p;
                    y.add(p, v + c);
                });
                y.store(out + c, 1.0f / l);
            }
        });
}

// ------------------------------------------------------------------------------------------
// dq: the forward kernel's walk with three products per tile (see pskv_bwd_mfma.hip).
// ------------------------------------------------------------------------------------------
constexpr int kBwdWaves = 8;

__device__ inline float dot_rows(const uintx4 (&x)[kKS], const uintx4 (&y)[kKS])
{
    float acc = 0.f;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc = __builtin_fmaf(__uint_as_float(x[ks][e] << 16), __uint_as_float(y[ks][e] << 16), acc);
            acc = __builtin_fmaf(__uint_as_float(x[ks][e] & 0xffff0000u), __uint_as_float(y[ks][e] & 0xffff0000u), acc);
        }
    return acc + __shfl_xor(acc, 32, 64);
}

template <typename VIS, typename KF>
__device__ inline void dq_tile(const floatx16 &s, const floatx16 &dp, float c, float lse2, float drow, VIS vis, KF kf, floatx16 (&dq)[kDT])
{
    float ds[16];
#pragma unroll
    for (int e = 0; e < 16; ++e)
        ds[e] = vis(e) ? fast_exp2(__builtin_fmaf(s[e], c, -lse2)) * (dp[e] - drow) : 0.f;
    // (The products as fp32 numbers, which split16 cuts into three: without the test the compiler would take each into the
    // first of its subtractions, and a key of a whole prefix tile weigh otherwise than of a ragged one or of a candidate's own.)
#pragma unroll
    for (int e = 0; e < 16; ++e)
        asm volatile("" : "+v"(ds[e]));
    const Split w = split16(ds);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) {
            const bf16x8 k = kf(dt, j);
#pragma unroll
            for (int part = kParts - 1; part >= 0; --part)
                dq[dt] = mma(k, w.p[part][j], dq[dt]);
        }
}

__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2)))
void hd64_bwd_dq_kernel(BwdArgs g, Spread sp)
{
    const Args &a = g.f;
    extern __shared__ __align__(256) unsigned char smem_generic[];
    lds_u8 *img = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X = make_hd64_ctx(a, tid);
    X.scr = img + sp.chunk * kTile + wave * kImg;
    const TilePlaces tp = tile_places(half_places(X.lane));
    const int nblocks = (X.Mtot + kBlockRows - 1) / kBlockRows, VH = a.Np * a.Hkv;
    bool bad = false;

    for (int vh = blockIdx.x % sp.vh_slots; vh < VH; vh += sp.vh_slots) {
        set_vhead(a, X, vh);
        const int T = (X.P + kTileKeys - 1) / kTileKeys;
        const bool resident = T <= sp.chunk;
        // (Nothing requested in between, as in the forward kernel: 48 candidates x 29 positions, P 206, 14/2 heads:
        // 27.4 us with the first block's rows asked for there, 26.1 so.)
        if (resident) {
            stage_request(a, X, img, 0, T, tid);
            stage_finish();
        }
        for (int it = 0; round_base(sp, kBwdWaves, it) < nblocks; ++it) {
            const int blk = round_base(sp, kBwdWaves, it) + wave;
            const bool has = blk < nblocks;
            const Rows x = make_rows(a, X, has ? blk : nblocks - 1);
            const bool work = has && __builtin_amdgcn_ballot_w64(x.valid) != 0;
            const int ri = x.valid ? x.i : 0; // padded rows take row 0 of their candidate and are stored as zero
            const float lse2 = a.lse[((long long)x.b * a.Hq + x.h) * a.S + ri] * kLog2e;
            uintx4 q[kKS], dof[kKS];
            float drow;
            {
                uintx4 of[kKS];
                const long long oo = (long long)x.b * a.o_sb + (long long)ri * a.o_ss + (long long)x.h * a.o_sh;
                load_row(a.q, (long long)x.b * a.q_sb + (long long)ri * a.q_ss + (long long)x.h * a.q_sh, X.h, q);
                load_row(g.dout, oo, X.h, dof);
                load_row(a.out, oo, X.h, of);
                drow = dot_rows(dof, of);
            }
            floatx16 dq[kDT];
#pragma unroll
            for (int dt = 0; dt < kDT; ++dt)
                dq[dt] = zero16();
            for (int t0 = 0; t0 < T; t0 += sp.chunk) {
                const int n = T - t0 < sp.chunk ? T - t0 : sp.chunk;
                if (!resident) {
                    stage_request(a, X, img, t0, n, tid);
                    stage_finish();
                }
                if (!work)
                    continue;
                auto tile = [&](int t, auto vis) __attribute__((always_inline)) {
                    lds_u8 *ki = img + t * kTile, *vi = ki + kImg;
                    floatx16 s = zero16(), dp = zero16();
#pragma unroll
                    for (int ks = 0; ks < kKS; ++ks) {
                        s = mma(tile_row_frag(tp, ki, ks), as_bf16x8(q[ks]), s);
                        dp = mma(tile_row_frag(tp, vi, ks), as_bf16x8(dof[ks]), dp);
                    }
                    dq_tile(s, dp, X.c, lse2, drow, vis, [&](int dt, int j) { return tile_col_frag(tp, ki, dt, j); }, dq);
                };
                // whole tiles, seen by every row, and the prefix's last, ragged one
                const int whole = X.P / kTileKeys - t0 < n ? X.P / kTileKeys - t0 : n;
                int t = 0;
                for (; t < whole; ++t)
                    tile(t, [](int) { return true; });
                if (t < n) {
                    const int nv = X.P - (t0 + t) * kTileKeys - 4 * X.h;
                    tile(t, [&](int e) { return 8 * (e >> 2) + (e & 3) < nv; });
                }
            }
            if (work) {
                const OwnList own = own_list(a, X, x);
                for (int k0 = 0; k0 < own.n; k0 += kTileKeys) {
                    const long long row = own_row(a, X, x, k0);
                    uintx4 kf[kKS], vf[kKS];
                    load_row(X.ksg, row, X.h, kf);
                    load_row(X.vsg, row, X.h, vf);
                    rows_to_image(X, X.scr, kf);
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    floatx16 s = zero16(), dp = zero16();
#pragma unroll
                    for (int ks = 0; ks < kKS; ++ks) {
                        s = mma(as_bf16x8(kf[ks]), as_bf16x8(q[ks]), s);
                        dp = mma(as_bf16x8(vf[ks]), as_bf16x8(dof[ks]), dp);
                    }
                    const int rel = k0 + 4 * X.h - own.first;
                    dq_tile(s, dp, X.c, lse2, drow, [&](int e) { return (unsigned)(rel + 8 * (e >> 2) + (e & 3)) <= (unsigned)x.i; },
                            [&](int dt, int j) { return frag_tr(X.scr, dt, j, X.lane); }, dq);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
            }
            if (has) {
                store_transposed(reinterpret_cast<unsigned short *>(g.dq) + (long long)x.b * a.q_sb + (long long)x.i * a.q_ss +
                                     (long long)x.h * a.q_sh,
                                 X.h, x.exists, x.valid, a.scale, dq);
                bad |= __builtin_amdgcn_ballot_w64(x.valid && has_nan(dq)) != 0;
            }
        }
    }
    if (bad)
        for_stored_rows(sp, kBwdWaves, tid, [](const Args &a, const Ctx &X, const Rows &x) {
            const BwdArgs &g = first_parameter<BwdArgs>();
            const long long at = (long long)x.b * a.q_sb + (long long)x.i * a.q_ss + (long long)x.h * a.q_sh;
            const long long oo = (long long)x.b * a.o_sb + (long long)x.i * a.o_ss + (long long)x.h * a.o_sh;
            unsigned short *dq = reinterpret_cast<unsigned short *>(g.dq) + at;
            const unsigned short *q = reinterpret_cast<const unsigned short *>(a.q) + at, *dout = reinterpret_cast<const unsigned short *>(g.dout) + oo;
            const float lse2 = a.lse[((long long)x.b * a.Hq + x.h) * a.S + x.i] * kLog2e;
            const float drow = lane_dot(dout, reinterpret_cast<const unsigned short *>(a.out) + oo);
#pragma unroll 1
            for (int c = 8 * X.h; c < kW; c += 16) {
                if (!to_form_anew(dq + c))
                    continue;
                Columns y;
                for_visible_keys(a, X, x, [&](const unsigned short *k, const unsigned short *v) {
                    y.add(fast_exp2(__builtin_fmaf(lane_dot(q, k), X.c, -lse2)) * (lane_dot(dout, v) - drow), k + c);
                });
                y.store(dq + c, a.scale);
            }
        });
}

// ------------------------------------------------------------------------------------------
// dk, dv: a workgroup of four wavefronts per (candidate, KV head, 32 suffix keys); the wavefronts take
// the 32-row blocks of the candidate's rows i*G + g in turn, a lane owning a key column
// (S = Q K^T, dP = dO V^T, then dV^T += dO^T P, dK^T += Q^T dS: see bwd_dkv_mfma_kernel), and are summed
// through LDS at the end.
// ------------------------------------------------------------------------------------------
constexpr int kDkvW = 4;
constexpr int kDkvScr = 2 * kImg + 512; // per wavefront: images of dO and Q, then lse, <dout,out>, position of the block's rows
constexpr int kDkvLds = kDkvW * 2 * kImg > kDkvW * kDkvScr ? kDkvW * 2 * kImg : kDkvW * kDkvScr;

__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2)))
void hd64_bwd_dkv_kernel(BwdArgs g, int nkt)
{
    const Args &a = g.f;
    extern __shared__ __align__(16) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    typedef __attribute__((address_space(3))) float lds_f32;
    typedef __attribute__((address_space(3))) floatx4 lds_f32x4;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const Ctx X = make_hd64_ctx(a, tid);
    const int unit = blockIdx.x / nkt, kt = blockIdx.x - unit * nkt;
    const int b = unit / a.Hkv, k = unit - b * a.Hkv;
    const int k0 = kt * kTileKeys, len = len_uniform(a, b), key = k0 + X.c32;
    lds_u8 *doi = smem + wave * kDkvScr, *qi = doi + kImg;
    lds_f32 *aux = (lds_f32 *)(qi + kImg);
    const long long koff = (long long)b * a.ks_sb + (long long)k * a.ks_sh;

    floatx16 dk[kDT], dv[kDT];
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt)
        dk[dt] = dv[dt] = zero16();
    if (k0 < len) {
        uintx4 kf[kKS], vf[kKS];
        const long long krow = koff + (long long)(key < len ? key : len - 1) * a.ks_ss;
        load_row(a.ks, krow, X.h, kf);
        load_row(a.vs, krow, X.h, vf);
        const long long qb = (long long)b * a.q_sb + (long long)k * a.G * a.q_sh, ob = (long long)b * a.o_sb + (long long)k * a.G * a.o_sh;
        const int nrows = len * a.G; // rows with i < len; those with i >= k0 can see a key of the tile
        for (int r0 = k0 * a.G / kBlockRows * kBlockRows + wave * kBlockRows; r0 < nrows; r0 += kDkvW * kBlockRows) {
            const int rl = r0 + X.c32 < nrows ? r0 + X.c32 : nrows - 1;
            const int i = (int)fdiv(rl, a.div_g), gq = rl - i * a.G;
            const long long oo = ob + (long long)i * a.o_ss + (long long)gq * a.o_sh;
            const float lse = a.lse[((long long)b * a.Hq + k * a.G + gq) * a.S + i];
            uintx4 q[kKS], dof[kKS];
            float drow;
            {
                uintx4 of[kKS];
                load_row(a.q, qb + (long long)i * a.q_ss + (long long)gq * a.q_sh, X.h, q);
                load_row(g.dout, oo, X.h, dof);
                load_row(a.out, oo, X.h, of);
                drow = dot_rows(dof, of);
            }
            rows_to_image(X, doi, dof);
            rows_to_image(X, qi, q);
            if (X.h == 0) {
                aux[X.c32] = lse * kLog2e;
                aux[32 + X.c32] = drow;
                aux[64 + X.c32] = r0 + X.c32 < nrows ? (float)i : -1.f;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            floatx16 s = zero16(), dp = zero16();
#pragma unroll
            for (int ks = 0; ks < kKS; ++ks) {
                s = mma(as_bf16x8(q[ks]), as_bf16x8(kf[ks]), s);
                dp = mma(as_bf16x8(dof[ks]), as_bf16x8(vf[ks]), dp);
            }
            float p[16], ds[16];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) { // element 4kk + t: row 8kk + 4h + t
                const floatx4 l4 = *(lds_f32x4 *)(aux + 8 * kk + 4 * X.h), d4 = *(lds_f32x4 *)(aux + 32 + 8 * kk + 4 * X.h),
                              i4 = *(lds_f32x4 *)(aux + 64 + 8 * kk + 4 * X.h);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int e = 4 * kk + t;
                    const bool vis = (float)key <= i4[t] && key < len;
                    p[e] = vis ? fast_exp2(__builtin_fmaf(s[e], X.c, -l4[t])) : 0.f;
                    ds[e] = p[e] * (dp[e] - d4[t]);
                }
            }
            const Split wp = split16(p), ws = split16(ds);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int dt = 0; dt < kDT; ++dt) {
                    const bf16x8 x = frag_tr(doi, dt, j, X.lane), y = frag_tr(qi, dt, j, X.lane);
#pragma unroll
                    for (int part = kParts - 1; part >= 0; --part) {
                        dv[dt] = mma(x, wp.p[part][j], dv[dt]);
                        dk[dt] = mma(y, ws.p[part][j], dk[dt]);
                    }
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    // Sum over the wavefronts, dk and then dv: wavefront w adds up and stores column tile w / 2, pieces of the
    // pair pr = w % 2 (elements 8pr .. 8pr + 7).
    const int dt = wave >> 1, pr = wave & 1;
    const long long at = koff + (long long)(key < a.S ? key : 0) * a.ks_ss;
    unsigned long long nan[2]; // lanes with a NaN among their sums
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        __syncthreads();
#pragma unroll
        for (int d = 0; d < kDT; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const floatx16 &v = which == 0 ? dk[d] : dv[d];
                *(lds_f32x4 *)(smem + ((wave * kDT + d) * 4 + i) * 1024 + X.lane * 16) = floatx4{v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]};
            }
        __syncthreads();
        floatx4 y[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int w = 0; w < kDkvW; ++w)
#pragma unroll
            for (int i = 0; i < 2; ++i)
                y[i] += *(lds_f32x4 *)(smem + ((w * kDT + dt) * 4 + 2 * pr + i) * 1024 + X.lane * 16);
        bool bad = false;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            bad |= y[0][t] != y[0][t] || y[1][t] != y[1][t];
        nan[which] = __builtin_amdgcn_ballot_w64(key < len && bad);
        const float f = which == 0 ? a.scale : 1.f;
        unsigned w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            w[i] = key < len ? pack_bf16(y[i >> 1][2 * (i & 1)] * f, y[i >> 1][2 * (i & 1) + 1] * f) : 0u;
        const auto u = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
        const auto v = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
        if (key < a.S)
            *reinterpret_cast<uintx4 *>(reinterpret_cast<unsigned short *>(which == 0 ? g.dk : g.dv) + at + 32 * dt + 16 * pr + 8 * X.h) =
                uintx4{u[0], v[0], u[1], v[1]};
    }
    // (see to_form_anew)
#pragma unroll 1
    for (int which = 0; which < 2; ++which) {
        if (!(((unsigned)(nan[which] | (nan[which] >> 32)) >> X.c32) & 1u))
            continue;
        const unsigned short *krow = reinterpret_cast<const unsigned short *>(a.ks) + at, *vrow = reinterpret_cast<const unsigned short *>(a.vs) + at;
        const int c = 32 * dt + 16 * pr + 8 * X.h;
        Columns y;
#pragma unroll 1
        for (int rl = key * a.G; rl < len * a.G; ++rl) { // the rows that see the key
            const int i = (int)fdiv(rl, a.div_g), h = k * a.G + rl - i * a.G;
            const long long oo = (long long)b * a.o_sb + (long long)i * a.o_ss + (long long)h * a.o_sh;
            const unsigned short *q = reinterpret_cast<const unsigned short *>(a.q) + (long long)b * a.q_sb + (long long)i * a.q_ss + (long long)h * a.q_sh;
            const unsigned short *dout = reinterpret_cast<const unsigned short *>(g.dout) + oo, *out = reinterpret_cast<const unsigned short *>(a.out) + oo;
            const float lse2 = a.lse[((long long)b * a.Hq + h) * a.S + i] * kLog2e;
            const float p = fast_exp2(__builtin_fmaf(lane_dot(q, krow), X.c, -lse2));
            y.add(which == 0 ? p * (lane_dot(dout, vrow) - lane_dot(dout, out)) : p, (which == 0 ? q : dout) + c);
        }
        y.store(reinterpret_cast<unsigned short *>(which == 0 ? g.dk : g.dv) + at + c, which == 0 ? a.scale : 1.f);
    }
}
static_assert(kDkvW == 2 * kDT && kDkvW * kDT * 4 * 1024 <= kDkvLds, "LDS of the final sum");

constexpr int kMaxLds = 160 * 1024;

int device_cu_count(hipError_t &e)
{
    static DeviceSlots cu_by_device;
    return device_setup_once(cu_by_device, e, [] {
        hipError_t s = hipFuncSetAttribute(reinterpret_cast<const void *>(hd64_fwd_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
        if (s == hipSuccess)
            s = hipFuncSetAttribute(reinterpret_cast<const void *>(hd64_bwd_dq_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
        return s;
    });
}

// Grid, LDS and chunk size for a walk with `waves` wavefronts per workgroup:
// half of a compute unit's LDS where the whole prefix fits into that (two workgroups per compute unit), all
// of it otherwise, in chunks if need be.
struct Shape {
    unsigned grid;
    size_t lds;
    Spread sp;
};
Shape make_shape(const Args &a, int num_cu, int waves, int most_per_cu)
{
    const int T = (a.P + kTileKeys - 1) / kTileKeys, tile = kTile, scratch = waves * kImg;
    const int half = (kMaxLds / 2 - scratch) / tile, whole = (kMaxLds - scratch) / tile;
    Shape s;
    const bool two = most_per_cu > 1 && T <= half;
    s.sp.chunk = T <= whole ? (T > 0 ? T : 1) : whole;
    s.lds = (size_t)s.sp.chunk * tile + scratch;
    const long long VH = (long long)a.Np * a.Hkv, slots = (long long)num_cu * (two ? 2 : 1);
    const long long nblocks = ((long long)a.C * a.S * a.G + kBlockRows - 1) / kBlockRows, useful = (nblocks + waves - 1) / waves;
    const long long vh_slots = VH < slots ? VH : slots;
    long long per_vh = slots / vh_slots;
    per_vh = per_vh < useful ? per_vh : useful;
    s.sp.per_vh = (int)per_vh;
    s.sp.vh_slots = (int)vh_slots;
    s.grid = (unsigned)(per_vh * vh_slots);
    return s;
}

} // namespace

bool hd64_supported(const Args &a, int dtype)
{
    return dtype == 1 && !a.plain && a.D == kW && (long long)a.C * a.S * a.G <= 0x7fffffffLL - kBlockRows;
}

bool hd64_dkv_supported(const Args &a, int dtype)
{
    return hd64_supported(a, dtype) && launch_fits((long long)a.B * a.Hkv * ((a.S + kTileKeys - 1) / kTileKeys), kDkvW * 64);
}

hipError_t launch_hd64_fwd(const Args &a, hipStream_t stream)
{
    hipError_t e;
    const int num_cu = device_cu_count(e);
    if (num_cu == 0)
        return e;
    const Shape s = make_shape(a, num_cu, kFwdWaves, 2);
    return launch_kernel(hd64_fwd_kernel, dim3(s.grid), dim3(kFwdWaves * 64), s.lds, stream, a, s.sp);
}

hipError_t launch_hd64_bwd_dq(const BwdArgs &g, hipStream_t stream)
{
    hipError_t e;
    const int num_cu = device_cu_count(e);
    if (num_cu == 0)
        return e;
    const Shape s = make_shape(g.f, num_cu, kBwdWaves, 1);
    return launch_kernel(hd64_bwd_dq_kernel, dim3(s.grid), dim3(kBwdWaves * 64), s.lds, stream, g, s.sp);
}

hipError_t launch_hd64_bwd_dkv(const BwdArgs &g, hipStream_t stream)
{
    const Args &a = g.f;
    const int nkt = (a.S + kTileKeys - 1) / kTileKeys;
    return launch_kernel(hd64_bwd_dkv_kernel, dim3((unsigned)((long long)a.B * a.Hkv * nkt)), dim3(kDkvW * 64), kDkvLds, stream, g, nkt);
}

} // namespace pskv
