// Matrix-core kernels for fp32 tensors (head dim 64 or 128): forward pass and the gradients of
// the suffix side, in double precision from the exactly widened inputs to the one final rounding,
// like the vector kernels of pskv_simple.hip and pskv_bwd_simple.hip.
//
// What bounds this path is double-precision arithmetic (72 TFLOP/s in a large library product, a
// nineteenth of what a bf16 one reaches), so everything here serves v_mfma_f64_16x16x4_f64 (64 cycles each): a
// wavefront owns 16 query rows (or 16 suffix keys) and meets 16 keys (rows) at a time, 4 KB or 8 KB
// of K and as much of V per 2000 to 4000 cycles of matrix work, which L1 and L2 deliver straight
// into registers: no staging of tiles, no barrier between them.  The vector kernels it takes the place
// of run one wavefront per query row with one multiply-add per loaded element and lane.  Backward pass
// of 16 candidates of 20 rows, 100 prefix rows, 32/8 heads of 128 columns: 197 us there, 46 us here (of
// which the matrix cores are busy 13; a wavefront has two or three tiles of its own, so what is left
// is the latency of its beginning and end and the odd tile).
//
// Operand layouts (lane l: c = l % 16, kq = l / 16).  A[16][4] and B[4][16] hold one double per lane,
// A[c][kq] and B[kq][c]; D[16][16] holds four, element r being D[4r + kq][c].
//     S^T[key][row] = sum_d K[key][d] Q[row][d]      the 4 d of one instruction are 16s + 4kq + e for
//                                                    kq = 0..3: a lane's d come in runs of 4 floats
//     O^T[d][row]  += sum_key V[key][d] P^T[key][row]   step r contracts the keys 4r + kq: element r
//                                                    of S^T is the B operand as it stands; row c of
//                                                    column tile dt is d = c*(D/16) + dt, so that a
//                                                    lane's V elements and results are runs as well
// The keys a block of rows meets form one list of 16-key tiles: the prefix, then the own suffix
// keys of every candidate the block touches.  The four wavefronts of a workgroup share one block:
// each takes every fourth tile, starting with another one from block to block so that no SIMD is
// always the one with the odd tile, and they are summed through LDS at the end.
//
// The matrix cores and the vector ALU share the double-precision units: widening both operands at
// every use costs a quarter of the time (82 instead of 64 cycles per matrix instruction, measured),
// so the operand that stays the same from tile to tile (the block's rows of q and dout; K and V for dk
// and dv) is widened once into LDS, from where all four wavefronts read it.
#include "pskv_internal.h"

namespace pskv {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kTR = 16;    // rows (or keys) of a tile
constexpr int kWaves = 4;  // wavefronts of a workgroup

__device__ inline unsigned fdiv(unsigned n, FastDiv d) { return (unsigned)(((unsigned long long)n * d.mul) >> d.shift); }
__device__ inline doublex4 mfma(double a, double b, doublex4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ inline doublex4 zero4() { return doublex4{0., 0., 0., 0.}; }

// Sum and maximum over the four lanes that share a column.
__device__ inline double sum_kq(double v)
{
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}
__device__ inline double max_kq(double v)
{
    v = fmax(v, __shfl_xor(v, 16, 64));
    return fmax(v, __shfl_xor(v, 32, 64));
}

template <int D> struct Frag { // a lane's quarter of a row: d = 16s + 4kq + e in v[s][e]
    floatx4 v[D / 16];
};
template <int D> struct Cols { // columns c*(D/16) .. of the rows 4r + kq, r = 0..3
    floatx4 v[4][D / 64];
};
template <int D> __device__ inline void load_frag(const float *row, int kq, Frag<D> &f)
{
#pragma unroll
    for (int s = 0; s < D / 16; ++s)
        f.v[s] = *reinterpret_cast<const floatx4 *>(row + 16 * s + 4 * kq);
}
template <int D> __device__ inline void load_cols(const float *row, int c, int r, Cols<D> &f)
{
#pragma unroll
    for (int i = 0; i < D / 64; ++i)
        f.v[r][i] = *reinterpret_cast<const floatx4 *>(row + c * (D / 16) + 4 * i);
}
typedef double doublex2 __attribute__((ext_vector_type(2)));

// A widened fragment in LDS: the pair of instruction pair i (d = 16s + 4kq + 2j, + 1 with i = 2s + j) at
// [i*64 + lane].
template <int D> constexpr size_t kWideBytes = (size_t)16 * D * sizeof(double);
template <int D> __device__ inline void widen_share(const float *row, int kq, int lane, int wave, doublex2 *wide)
{
#pragma unroll
    for (int t = 0; t < D / 64; ++t) { // a quarter of the fragment per wavefront
        const int s = wave * (D / 64) + t;
        const floatx4 v = *reinterpret_cast<const floatx4 *>(row + 16 * s + 4 * kq);
        wide[(2 * s) * 64 + lane] = doublex2{(double)v[0], (double)v[1]};
        wide[(2 * s + 1) * 64 + lane] = doublex2{(double)v[2], (double)v[3]};
    }
}
template <int D> __device__ inline doublex4 contract(const Frag<D> &a, const doublex2 *wide, int lane)
{
    // two chains, so that an instruction does not wait for the one before it
    doublex4 x = zero4(), y = zero4();
#pragma unroll
    for (int s = 0; s < D / 16; ++s) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const doublex2 b = wide[(2 * s + j) * 64 + lane];
            x = mfma((double)a.v[s][2 * j], b[0], x);
            y = mfma((double)a.v[s][2 * j + 1], b[1], y);
        }
        if constexpr (D > 64) // widen a few operands at a time (the empty statement makes the sums exist here)
            asm volatile("" : "+v"(x), "+v"(y));
    }
    return x + y;
}
// acc[dt] += cols^T p: the second products
template <int D> __device__ inline void accumulate(const Cols<D> &cols, const doublex4 &p, doublex4 (&acc)[D / 16])
{
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt)
            acc[dt] = mfma((double)cols.v[r][dt / 4][dt % 4], p[r], acc[dt]);
        if constexpr (D > 64)
            __builtin_amdgcn_sched_barrier(0);
    }
}

__device__ inline int clamp_to(int n, int most) { return n < 0 ? 0 : (n > most ? most : n); }
__device__ inline int length_of(const Args &a, int b) { return a.len ? clamp_to(a.len[b], a.S) : a.S; }

// An entry of an index array that the whole wavefront asks for: through the constant address space (the
// array is not written during the call), which makes it a scalar load and what follows from it scalar.
__device__ inline int uniform_entry(const int *p, int i)
{
    typedef const __attribute__((address_space(4))) int *const_int_ptr;
    return ((const_int_ptr)(unsigned long long)p)[__builtin_amdgcn_readfirstlane(i)];
}
__device__ inline int uniform_length(const Args &a, int b) { return a.len ? clamp_to(uniform_entry(a.len, b), a.S) : a.S; }

// A block of 16 stacked rows r = (b*S + i)*G + g of one (instruction, KV head) pair.
struct Block {
    int n, k;             // instruction, KV head
    int P;                // real prefix rows of the instruction
    long long pre;        // offset of the first of them
    int tok0, tok1;       // first and last token (candidate * S + position) of the block
    int b, i, h;          // the lane's own row: candidate, position, query head
    bool valid, exists;
    int ntp;              // prefix tiles
};

__device__ inline Block make_block(const Args &a, int vh, int blk, int c)
{
    Block x;
    x.n = vh / a.Hkv;
    x.k = vh - x.n * a.Hkv;
    x.P = a.plen ? clamp_to(uniform_entry(a.plen, x.n), a.P) : a.P;
    x.pre = (long long)x.n * a.kp_sn + (long long)(a.P - x.P) * a.kp_sp + (long long)x.k * a.kp_sh;
    x.ntp = (x.P + kTR - 1) / kTR;
    const int M = a.C * a.S * a.G, r0 = blk * kTR;
    const int last = r0 + kTR - 1 < M ? r0 + kTR - 1 : M - 1;
    x.tok0 = (int)fdiv(r0, a.div_g);
    x.tok1 = (int)fdiv(last, a.div_g);
    const int r = r0 + c < M ? r0 + c : M - 1;
    x.exists = r0 + c < M;
    const int tok = (int)fdiv(r, a.div_g), bl = (int)fdiv(tok, a.div_s);
    x.b = x.n * a.C + bl;
    x.i = tok - bl * a.S;
    x.h = x.k * a.G + (r - tok * a.G);
    x.valid = x.exists && x.i < length_of(a, x.b);
    return x;
}

// Key tile u of the block's list: the rows, and the last of its keys that the lane's row sees.
struct Tile {
    const float *k, *v; // row 0
    long long stride;
    int key0, last;     // first key, last key that exists for the block (rows beyond it are never read)
    int lim;
};

__device__ inline bool make_tile(const Args &a, const Block &x, int u, Tile &t)
{
    if (u < x.ntp) {
        t.k = reinterpret_cast<const float *>(a.kp) + x.pre;
        t.v = reinterpret_cast<const float *>(a.vp) + x.pre;
        t.stride = a.kp_sp;
        t.key0 = u * kTR;
        t.last = t.lim = x.P - 1;
        return true;
    }
    u -= x.ntp;
    const int bl1 = (int)fdiv(x.tok1, a.div_s);
    for (int bl = (int)fdiv(x.tok0, a.div_s); bl <= bl1; ++bl) {
        const int b = x.n * a.C + bl, len = uniform_length(a, b);
        const int lo = x.tok0 - bl * a.S > 0 ? x.tok0 - bl * a.S : 0;
        const int hi = x.tok1 - bl * a.S < len - 1 ? x.tok1 - bl * a.S : len - 1; // last key any row of the block sees
        if (lo >= len)
            continue;
        const int tiles = hi / kTR + 1;
        if (u < tiles) {
            const long long off = (long long)b * a.ks_sb + (long long)x.k * a.ks_sh;
            t.k = reinterpret_cast<const float *>(a.ks) + off;
            t.v = reinterpret_cast<const float *>(a.vs) + off;
            t.stride = a.ks_ss;
            t.key0 = u * kTR;
            t.last = hi;
            t.lim = x.b == b ? x.i : -1;
            return true;
        }
        u -= tiles;
    }
    return false;
}

__device__ inline long long tile_row(const Tile &t, int j)
{
    const int key = t.key0 + j;
    return (long long)(key < t.last ? key : t.last) * t.stride;
}

// The four wavefronts' accumulators, each scaled by its `f`, summed, scaled by `inv` and stored at `row`
// (zeros when not valid): wavefront w takes the elements r = w.  64 columns at a time, so that the
// buffer (kGatherBytes, free when this is called) is no larger than what the tiles needed.
//
// Returns whether one of the lane's sums is NaN in a valid row: see finish_alone.
constexpr size_t kGatherBytes = (size_t)kWaves * 4 * 4 * 64 * sizeof(double);
template <int D>
__device__ inline bool gather_store(double *buf, int wave, int lane, const doublex4 (&x)[D / 16], double f, float *row, double inv,
                                    bool exists, bool valid)
{
    bool nan = false;
    row += (4 * wave + (lane >> 4)) * (D / 16); // the run of columns of element r = wave
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
        if (i > 0)
            __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                buf[((wave * 4 + r) * 4 + j) * 64 + lane] = x[4 * i + j][r] * f;
        __syncthreads();
        doublex4 sum = zero4();
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int w = 0; w < kWaves; ++w)
                sum[j] += buf[((w * 4 + wave) * 4 + j) * 64 + lane];
        floatx4 y;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            y[j] = valid ? (float)(sum[j] * inv) : 0.f;
        nan |= y[0] != y[0] || y[1] != y[1] || y[2] != y[2] || y[3] != y[3];
        if (exists)
            *reinterpret_cast<floatx4 *>(row + 4 * i) = y;
    }
    return nan;
}

// The products take hidden terms - another candidate's keys, keys behind the row's position - with a weight
// of zero, and zero times an infinity or NaN among them is NaN.  That is all such a term can do (the
// scores are replaced before anything is made of them), so a lane that finds a NaN among its sums
// forms those columns anew, alone, from the terms that its row has, and stores them over the others:
// each(term) calls term(weight, row) for these.  Kept behind the last use of the accumulators: no
// registers are held for it, and a row without NaN pays a comparison.
template <int D> __device__ inline double lane_dot(const float *x, const float *y)
{
    double acc = 0.;
#pragma unroll 4
    for (int d = 0; d < D; ++d)
        acc += (double)x[d] * (double)y[d];
    return acc;
}
template <int D, typename F> __device__ inline void finish_alone(int wave, int lane, float *row, double inv, F each)
{
    asm volatile("" : "+v"(lane)); // (nothing of this is worked out ahead)
    const int col = (4 * wave + (lane >> 4)) * (D / 16);
    for (int c0 = col; c0 < col + D / 16; c0 += 4) {
        doublex4 sum = zero4();
        each([&](double w, const float *r) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                sum[j] += w * (double)r[c0 + j];
        });
#pragma unroll
        for (int j = 0; j < 4; ++j)
            row[c0 + j] = (float)(sum[j] * inv);
    }
}
// Calls f(K row, V row) for the keys that the lane's row sees.
template <typename F> __device__ inline void for_visible_keys(const Args &a, const Block &x, F f)
{
    const float *kp = reinterpret_cast<const float *>(a.kp) + x.pre, *vp = reinterpret_cast<const float *>(a.vp) + x.pre;
    for (int j = 0; j < x.P; ++j)
        f(kp + (long long)j * a.kp_sp, vp + (long long)j * a.kp_sp);
    const long long own = (long long)x.b * a.ks_sb + (long long)x.k * a.ks_sh;
    const float *ks = reinterpret_cast<const float *>(a.ks) + own, *vs = reinterpret_cast<const float *>(a.vs) + own;
    for (int j = 0; j <= x.i; ++j)
        f(ks + (long long)j * a.ks_ss, vs + (long long)j * a.ks_ss);
}

template <int D>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2)))
void f32_fwd_kernel(Args a_, int nblk)
{
    const Args &a = a_;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, kq = lane >> 4;
    const int vh = blockIdx.x / nblk, blk = blockIdx.x - vh * nblk;
    const Block x = make_block(a, vh, blk, c);
    doublex2 *qw = reinterpret_cast<doublex2 *>(smem_raw);
    double *buf = reinterpret_cast<double *>(smem_raw), *st = reinterpret_cast<double *>(smem_raw + kGatherBytes);

    doublex4 o[D / 16];
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
        o[dt] = zero4();
    double m = -INFINITY, l = 0.;
    if (__builtin_amdgcn_ballot_w64(x.valid) != 0) { // the same for all four wavefronts
        int u = (wave + blk) & (kWaves - 1);
        Tile t;
        bool more = make_tile(a, x, u, t);
        Frag<D> kf;
        if (more)
            load_frag<D>(t.k + tile_row(t, c), kq, kf);
        // padded rows take row 0 of their candidate: whatever it holds stays in their own column
        widen_share<D>(reinterpret_cast<const float *>(a.q) + (long long)x.b * a.q_sb + (long long)(x.valid ? x.i : 0) * a.q_ss +
                           (long long)x.h * a.q_sh,
                       kq, lane, wave, qw);
        __syncthreads();
        while (more) {
            Cols<D> vc;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                load_cols<D>(t.v + tile_row(t, 4 * r + kq), c, r, vc);
            doublex4 s = contract<D>(kf, qw, lane);
            const int lim = t.lim - t.key0 - kq;
            u += kWaves;
            more = make_tile(a, x, u, t);
            // The next tile's keys are on their way during the rest of this one (behind the last tile: the same
            // ones again; a load under a branch would have to be waited for where the branches meet).
            load_frag<D>(t.k + tile_row(t, c), kq, kf);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                s[r] = 4 * r <= lim ? s[r] * (double)a.scale : -INFINITY;
            const double mx = fmax(m, max_kq(fmax(fmax(s[0], s[1]), fmax(s[2], s[3]))));
            const double ref = mx == -INFINITY ? 0. : mx; // nothing visible yet: all weights zero
            if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
                const double alpha = exp(m - ref);
                l *= alpha;
#pragma unroll
                for (int dt = 0; dt < D / 16; ++dt)
                    o[dt] *= alpha;
                m = mx;
            }
            doublex4 p;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                p[r] = exp(s[r] - ref);
                l += p[r];
            }
            accumulate<D>(vc, p, o);
        }
    }
    l = sum_kq(l);
    if (kq == 0) {
        st[wave * 32 + c] = m;
        st[wave * 32 + 16 + c] = l;
    }
    __syncthreads();
    double top = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
        top = fmax(top, st[w * 32 + c]);
    double sum = 0.;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
        sum += st[w * 32 + 16 + c] * exp(st[w * 32 + c] - top);
    float *out = reinterpret_cast<float *>(a.out) + (long long)x.b * a.o_sb + (long long)x.i * a.o_ss + (long long)x.h * a.o_sh;
    const bool nan = gather_store<D>(buf, wave, lane, o, exp(m - top), out, 1. / sum, x.exists, x.valid);
    if (x.exists && a.lse && kq == 0 && wave == 0)
        a.lse[((long long)x.b * a.Hq + x.h) * a.S + x.i] = x.valid ? (float)(top + log(sum)) : -INFINITY;
    // (128 columns: the arguments are loaded anew there, as holding them costs the tiles scalar registers: 8 candidates x 34
    // positions, P 253, 8/2 heads: 20.1 us, 19.7 so, 19.6 without the check; for 64 columns, and in the backward pass, the
    // loads cost 1 to 3 % more than they save.)
    if (nan)
        finish_alone<D>(wave, lane, out, 1. / sum, [&](auto term) {
            const Args &a = D == 128 ? first_parameter<Args>() : a_;
            const float *q = reinterpret_cast<const float *>(a.q) + (long long)x.b * a.q_sb + (long long)x.i * a.q_ss + (long long)x.h * a.q_sh;
            for_visible_keys(a, x, [&](const float *k, const float *v) { term(exp(lane_dot<D>(q, k) * (double)a.scale - top), v); });
        });
}

// ------------------------------------------------------------------------------------------
// Gradients: p_j = exp(s_j - lse), dp_j = <dout_row, V_j>, ds_j = p_j (dp_j - <dout_row, out_row>),
//     dq_row = scale sum_j ds_j K_j,  dK_j = scale sum_rows ds_j q_row,  dV_j = sum_rows p_j dout_row.
// dq: blocks and key tiles of the forward pass.  dk, dv: a workgroup per (candidate, KV head, 16
// suffix keys), its wavefronts taking the 16-row tiles of the candidate's rows in turn.
// ------------------------------------------------------------------------------------------
template <int D> __device__ inline double dot_rows(const float *x, const float *y, int kq)
{
    double acc = 0.;
#pragma unroll
    for (int s = 0; s < D / 16; ++s) {
        const floatx4 u = *reinterpret_cast<const floatx4 *>(x + 16 * s + 4 * kq), v = *reinterpret_cast<const floatx4 *>(y + 16 * s + 4 * kq);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            acc += (double)u[e] * (double)v[e];
    }
    return sum_kq(acc);
}

template <int D> __device__ __attribute__((always_inline)) void dq_block(const BwdArgs &g, int nblk, int id, unsigned char *smem)
{
    const Args &a = g.f;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, kq = lane >> 4;
    const int vh = id / nblk, blk = id - vh * nblk;
    const Block x = make_block(a, vh, blk, c);
    doublex2 *qw = reinterpret_cast<doublex2 *>(smem), *dow = reinterpret_cast<doublex2 *>(smem + kWideBytes<D>);
    const long long row = (long long)x.b * a.q_sb + (long long)x.h * a.q_sh, orow = (long long)x.b * a.o_sb + (long long)x.h * a.o_sh;
    doublex4 dq[D / 16];
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
        dq[dt] = zero4();
    if (__builtin_amdgcn_ballot_w64(x.valid) != 0) {
        const int i = x.valid ? x.i : 0;
        int u = (wave + blk) & (kWaves - 1);
        Tile t;
        bool more = make_tile(a, x, u, t);
        Frag<D> kf, vf;
        if (more)
            load_frag<D>(t.k + tile_row(t, c), kq, kf);
        const float *dout = reinterpret_cast<const float *>(g.dout) + orow + (long long)i * a.o_ss;
        widen_share<D>(reinterpret_cast<const float *>(a.q) + row + (long long)i * a.q_ss, kq, lane, wave, qw);
        widen_share<D>(dout, kq, lane, wave, dow);
        const double lse = (double)a.lse[((long long)x.b * a.Hq + x.h) * a.S + i];
        const double drow = dot_rows<D>(dout, reinterpret_cast<const float *>(a.out) + orow + (long long)i * a.o_ss, kq);
        __syncthreads();
        while (more) {
            // each operand is requested one product ahead of its use
            load_frag<D>(t.v + tile_row(t, c), kq, vf);
            const doublex4 s = contract<D>(kf, qw, lane);
            __builtin_amdgcn_sched_barrier(0);
            Cols<D> kc;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                load_cols<D>(t.k + tile_row(t, 4 * r + kq), c, r, kc);
            const doublex4 dp = contract<D>(vf, dow, lane);
            __builtin_amdgcn_sched_barrier(0);
            const int lim = t.lim - t.key0 - kq;
            u += kWaves;
            more = make_tile(a, x, u, t);
            load_frag<D>(t.k + tile_row(t, c), kq, kf);
            doublex4 ds;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                ds[r] = exp(4 * r <= lim ? s[r] * (double)a.scale - lse : -INFINITY) * (dp[r] - drow);
            accumulate<D>(kc, ds, dq);
        }
    }
    __syncthreads(); // nobody reads q and dout any more: their place is free
    float *dst = reinterpret_cast<float *>(g.dq) + row + (long long)x.i * a.q_ss;
    if (gather_store<D>(reinterpret_cast<double *>(smem), wave, lane, dq, 1., dst, (double)a.scale, x.exists, x.valid))
        finish_alone<D>(wave, lane, dst, (double)a.scale, [&](auto term) {
            const long long at = orow + (long long)x.i * a.o_ss;
            const float *q = reinterpret_cast<const float *>(a.q) + row + (long long)x.i * a.q_ss, *dout = reinterpret_cast<const float *>(g.dout) + at;
            const double lse = (double)a.lse[((long long)x.b * a.Hq + x.h) * a.S + x.i];
            const double drow = lane_dot<D>(dout, reinterpret_cast<const float *>(a.out) + at);
            for_visible_keys(a, x, [&](const float *k, const float *v) {
                term(exp(lane_dot<D>(q, k) * (double)a.scale - lse) * (lane_dot<D>(dout, v) - drow), k);
            });
        });
}

template <int D> __device__ __attribute__((always_inline)) void dkv_unit(const BwdArgs &g, int nkt, int id, unsigned char *smem)
{
    const Args &a = g.f;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 15, kq = lane >> 4;
    const int unit = id / nkt, kt = id - unit * nkt;
    const int b = unit / a.Hkv, k = unit - b * a.Hkv;
    const int k0 = kt * kTR, len = uniform_length(a, b), key = k0 + c;
    const long long koff = (long long)b * a.ks_sb + (long long)k * a.ks_sh;
    doublex2 *kw = reinterpret_cast<doublex2 *>(smem), *vw = reinterpret_cast<doublex2 *>(smem + kWideBytes<D>);
    doublex4 dk[D / 16], dv[D / 16];
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
        dk[dt] = dv[dt] = zero4();
    if (k0 < len) {
        const long long krow = koff + (long long)(key < len ? key : len - 1) * a.ks_ss;
        widen_share<D>(reinterpret_cast<const float *>(a.ks) + krow, kq, lane, wave, kw);
        widen_share<D>(reinterpret_cast<const float *>(a.vs) + krow, kq, lane, wave, vw);
        __syncthreads();
        const long long qb = (long long)b * a.q_sb + (long long)k * a.G * a.q_sh, ob = (long long)b * a.o_sb + (long long)k * a.G * a.o_sh;
        const float *q = reinterpret_cast<const float *>(a.q) + qb;
        const float *dout = reinterpret_cast<const float *>(g.dout) + ob, *out = reinterpret_cast<const float *>(a.out) + ob;
        const int nrows = len * a.G; // rows i*G + g with i < len; those with i >= k0 can see a key of the tile
        const int first = k0 * a.G / kTR * kTR + ((wave + unit) & (kWaves - 1)) * kTR;
        for (int r0 = first; r0 < nrows; r0 += kWaves * kTR) {
            // row j of the tile, clamped into the candidate
            auto pos = [&](int j, int &i, int &gq) {
                const int rl = r0 + j < nrows ? r0 + j : nrows - 1;
                i = (int)fdiv(rl, a.div_g);
                gq = rl - i * a.G;
            };
            doublex4 s, dp;
            double lse_c, drow_c;
            {
                int i, gq;
                pos(c, i, gq);
                Frag<D> f;
                load_frag<D>(q + (long long)i * a.q_ss + (long long)gq * a.q_sh, kq, f);
                s = contract<D>(f, kw, lane);
                __builtin_amdgcn_sched_barrier(0);
                const long long oo = (long long)i * a.o_ss + (long long)gq * a.o_sh;
                load_frag<D>(dout + oo, kq, f);
                dp = contract<D>(f, vw, lane);
                lse_c = (double)a.lse[((long long)b * a.Hq + k * a.G + gq) * a.S + i];
                drow_c = dot_rows<D>(dout + oo, out + oo, kq);
            }
            Cols<D> qc, doc;
            doublex4 p, ds;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int i, gq;
                pos(4 * r + kq, i, gq);
                load_cols<D>(q + (long long)i * a.q_ss + (long long)gq * a.q_sh, c, r, qc);
                load_cols<D>(dout + (long long)i * a.o_ss + (long long)gq * a.o_sh, c, r, doc);
                const double lse = __shfl(lse_c, 4 * r + kq, 64), drow = __shfl(drow_c, 4 * r + kq, 64);
                const bool vis = r0 + 4 * r + kq < nrows && key <= i && key < len;
                p[r] = exp(vis ? s[r] * (double)a.scale - lse : -INFINITY);
                ds[r] = p[r] * (dp[r] - drow);
            }
            accumulate<D>(doc, p, dv);
            accumulate<D>(qc, ds, dk);
        }
    }
    double *buf = reinterpret_cast<double *>(smem);
    const long long at = koff + (long long)(key < a.S ? key : 0) * a.ks_ss;
    float *dst_k = reinterpret_cast<float *>(g.dk) + at, *dst_v = reinterpret_cast<float *>(g.dv) + at;
    __syncthreads();
    const bool nan_k = gather_store<D>(buf, wave, lane, dk, 1., dst_k, (double)a.scale, key < a.S, key < len);
    __syncthreads();
    const bool nan_v = gather_store<D>(buf, wave, lane, dv, 1., dst_v, 1., key < a.S, key < len);
    // the rows that see the lane's key
    auto for_rows = [&](auto f) {
        const float *kr = reinterpret_cast<const float *>(a.ks) + at, *vr = reinterpret_cast<const float *>(a.vs) + at;
        for (int rl = key * a.G; rl < len * a.G; ++rl) {
            const int i = (int)fdiv(rl, a.div_g), h = k * a.G + rl - i * a.G;
            const long long oo = (long long)b * a.o_sb + (long long)i * a.o_ss + (long long)h * a.o_sh;
            const float *q = reinterpret_cast<const float *>(a.q) + (long long)b * a.q_sb + (long long)i * a.q_ss + (long long)h * a.q_sh;
            const float *dout = reinterpret_cast<const float *>(g.dout) + oo, *out = reinterpret_cast<const float *>(a.out) + oo;
            f(q, dout, out, exp(lane_dot<D>(q, kr) * (double)a.scale - (double)a.lse[((long long)b * a.Hq + h) * a.S + i]), vr);
        }
    };
    if (nan_k)
        finish_alone<D>(wave, lane, dst_k, (double)a.scale, [&](auto term) {
            for_rows([&](const float *q, const float *dout, const float *out, double p, const float *vr) {
                term(p * (lane_dot<D>(dout, vr) - lane_dot<D>(dout, out)), q);
            });
        });
    if (nan_v)
        finish_alone<D>(wave, lane, dst_v, 1., [&](auto term) {
            for_rows([&](const float *, const float *dout, const float *, double p, const float *) { term(p, dout); });
        });
}

// One launch for all three gradients, neither of which needs anything of the other's: the dk/dv units,
// which take longer, first, and the dq blocks fill the chip round them.
template <int D>
__global__ __attribute__((amdgpu_flat_work_group_size(256, 256), amdgpu_waves_per_eu(2)))
void f32_bwd_kernel(BwdArgs g, int nblk, int nkt, int nunits)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if ((int)blockIdx.x < nunits)
        dkv_unit<D>(g, nkt, blockIdx.x, smem_raw);
    else
        dq_block<D>(g, nblk, blockIdx.x - nunits, smem_raw);
}

// (Two widened fragments of 128 columns, or the sums: 32 KB, under the limit that needs raising.)
static_assert(2 * kWideBytes<128> <= kGatherBytes && kGatherBytes + kWaves * 256 <= 64 * 1024, "LDS layout");
constexpr size_t kFwdLdsBytes = kGatherBytes + kWaves * 32 * sizeof(double), kBwdLdsBytes = kGatherBytes;

constexpr int kThreads = kWaves * 64;

// Blocks of rows, and dk/dv units, of all (instruction, KV head) pairs.
long long blocks_per_head(const Args &a) { return ((long long)a.C * a.S * a.G + kTR - 1) / kTR; }
long long all_blocks(const Args &a) { return blocks_per_head(a) * a.Np * a.Hkv; }
long long all_units(const Args &a) { return (long long)a.B * a.Hkv * ((a.S + kTR - 1) / kTR); }

} // namespace

bool f32_fwd_supported(const Args &a, int dtype)
{
    return dtype == 0 && !a.plain && (a.D == 64 || a.D == 128) && launch_fits(all_blocks(a), kThreads);
}
bool f32_bwd_supported(const Args &a, int dtype)
{
    return dtype == 0 && !a.plain && (a.D == 64 || a.D == 128) && launch_fits(all_units(a) + all_blocks(a), kThreads);
}

hipError_t launch_f32_fwd(const Args &a, hipStream_t stream)
{
    const dim3 grid((unsigned)all_blocks(a));
    const int nblk = (int)blocks_per_head(a);
    if (a.D == 64)
        return launch_kernel(f32_fwd_kernel<64>, grid, dim3(kThreads), kFwdLdsBytes, stream, a, nblk);
    return launch_kernel(f32_fwd_kernel<128>, grid, dim3(kThreads), kFwdLdsBytes, stream, a, nblk);
}

hipError_t launch_f32_bwd(const BwdArgs &g, hipStream_t stream)
{
    const Args &a = g.f;
    const int nblk = (int)blocks_per_head(a), nkt = (a.S + kTR - 1) / kTR, nunits = (int)all_units(a);
    const dim3 grid((unsigned)(all_units(a) + all_blocks(a)));
    if (a.D == 64)
        return launch_kernel(f32_bwd_kernel<64>, grid, dim3(kThreads), kBwdLdsBytes, stream, g, nblk, nkt, nunits);
    return launch_kernel(f32_bwd_kernel<128>, grid, dim3(kThreads), kBwdLdsBytes, stream, g, nblk, nkt, nunits);
}

} // namespace pskv
