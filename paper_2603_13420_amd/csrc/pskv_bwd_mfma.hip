// Matrix-core kernel for the query gradient of batched candidate-suffix attention on gfx950
// (bf16 tensors, head dim 128, prefix of any length - one shared prefix or one per instruction of
// the batched multi-instruction form -, any suffix shape).
//
// For a query row with softmax weights p_j = exp(s_j - lse) over its visible rows
// (prefix, then own suffix rows 0..i; derivative of Eq. 2, prefix K/V constant):
//     dp_j = <dout_row, V_j>,   ds_j = p_j (dp_j - <dout_row, out_row>),   dq_row = scale * sum_j ds_j K_j.
// Work is laid out as in the streamed forward kernels: a pass is one (KV head, group of 256
// stacked rows r = (b*S + i)*G + g) pair, each of the 8 wavefronts of a workgroup owns one
// 32-row block, and the prefix goes through LDS tile by tile (32 keys), double-buffered, one
// barrier per tile, read from HBM once and used by all 256 rows.  Per tile and block, with the
// transposed formulation of pskv_mfma.hpp (a lane owns one query column):
//     S^T  = K Q^T        A = K fragment (row-major image),   B = Q fragment
//     dP^T = V dO^T       A = V fragment (row-major image),   B = dO fragment
//     dS^T = P^T o (dP^T - D)                                 vector ALU, P^T = exp2(c S^T - lse)
//     dQ^T += K^T dS^T    A = K^T fragment (transposing image), B = dS^T packed to bf16
// so a slot of the LDS ring holds three 8 KB images: K and V row-major, K once more in the
// layout the transposing read wants.  The suffix rows of the block's own candidate(s) follow,
// with K/V fragments straight from global memory and K^T through the per-wave scratch tile.
// No running maximum is needed: lse comes from the forward pass, every weight is at most one.
// Two kernels further down serve candidates whose rows fill their own blocks well, with the prefix
// streamed or resident in LDS; this one takes what is left.
#include "pskv_packed.hpp"
#include <type_traits>

// Scratch of the entry point that allocates nothing (pskv_attn_bwd_noalloc): <dout_row, out_row> of
// every query row, B*Hq*S floats, handed from the dq kernel to the dk/dv kernel.  In host code this
// name is a stand-in for the symbol, not a device address: the address comes from
// hipGetSymbolAddress (noalloc_scratch() at the end of this file) and is what the kernels are given.
static __device__ __align__(256) unsigned char scratch[pskv::kNoAllocScratchBytes];

namespace pskv {
namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kBwdSlotBytes = 3 * kTileBytes;
constexpr int kBwdLdsBytes = 2 * kBwdSlotBytes + kNW * kScrBytes;
constexpr int kBwdPassRows = kNW * kBlockRows;

// Rows of a [.,.,H,D] tensor laid out like out (dout, out): lane (row c32, half h) gets
// d = 16*ks + 8*h ..+7 for ks = 0..7, as load_q does for q.
__device__ inline void load_o_like(const Args &a, const Ctx &X, const Row &x, const void *base, uintx4 (&dst)[8])
{
    const unsigned short *r = reinterpret_cast<const unsigned short *>(base) + (long long)x.rb * a.o_sb +
                              (long long)x.ri * a.o_ss + (long long)x.rh * a.o_sh + 8 * X.h;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
        dst[ks] = ld_global16(r + 16 * ks);
}

// Where <dout_row, out_row> of query row (candidate b, query head rh, suffix position ri) sits in
// the workspace: in the order of the stacked rows of its KV head, ((b*Hkv + k)*S + ri)*G + g, so
// that the 32 rows of a block are 128 contiguous bytes for the kernel that writes them and for
// the one that reads them back.
__device__ inline long long delta_index(const Args &a, long long b, int rh, int ri)
{
    const int k = (int)fdiv((unsigned)rh, a.div_g), gq = rh - k * a.G;
    return ((b * a.Hkv + k) * a.S + ri) * a.G + gq;
}

__device__ inline float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(unsigned w) { return __uint_as_float(w & 0xffff0000u); }

// <dout_row, out_row> is formed in the same order by every kernel, so that the dk/dv kernel finds the
// same bits whether it is handed the numbers or forms them itself: 8-column chunks one by one, then
// chunks c and c^1, then c^2, then c^4 of each half of the columns, then the halves.
__device__ inline float chunk_dot(uintx4 x, uintx4 y)
{
    float acc = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        acc = __builtin_fmaf(bf16_lo(x[e]), bf16_lo(y[e]), acc);
        acc = __builtin_fmaf(bf16_hi(x[e]), bf16_hi(y[e]), acc);
    }
    return acc;
}

// Sum over 8 neighbouring lanes (in every one of them), neighbours first.
__device__ inline float sum8(float v)
{
    auto dpp = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v += dpp(v, std::integral_constant<int, 0xB1>{});  // lane ^ 1
    v += dpp(v, std::integral_constant<int, 0x4E>{});  // lane ^ 2
    v += dpp(v, std::integral_constant<int, 0x141>{}); // the other four of the eight (all alike by now)
    return v;
}

// ... of the lane's row from the row's fragments (lane half h holds columns 16*ks + 8*h ..+7 of fragment ks).
__device__ inline float half_dot(const uintx4 (&x)[8], const uintx4 (&y)[8], int half)
{
    float p[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        p[i] = chunk_dot(x[4 * half + i], y[4 * half + i]);
        p[i] += __shfl_xor(p[i], 32, 64);
    }
    return (p[0] + p[1]) + (p[2] + p[3]);
}
__device__ inline float dout_dot_out(const uintx4 (&dof)[8], const uintx4 (&of)[8])
{
    return half_dot(dof, of, 0) + half_dot(dof, of, 1);
}

// dS^T of one 32-key tile from its raw scores s and dp; element e is visible iff vis(e).
// Returns the two B fragments (keys 0..15, 16..31) of the following product.
template <typename VIS>
__device__ inline void ds_tile(const floatx16 &s, const floatx16 &dp, float c, float lse2, float drow, VIS vis,
                               bf16x8 (&pf)[2])
{
    float ds[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const float p = vis(e) ? fast_exp2(__builtin_fmaf(s[e], c, -lse2)) : 0.f;
        ds[e] = p * (dp[e] - drow);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        uintx4 w = {pack_bf16(ds[8 * j + 0], ds[8 * j + 1]), pack_bf16(ds[8 * j + 2], ds[8 * j + 3]),
                    pack_bf16(ds[8 * j + 4], ds[8 * j + 5]), pack_bf16(ds[8 * j + 6], ds[8 * j + 7])};
        pf[j] = as_bf16x8(w);
    }
}

// O^T-style accumulation for the 16-key step j of a 32-key tile whose rows the lanes hold as
// row-major fragments (lane (key c32, half h): columns 16*ks + 8*h ..+7 in frag[ks]): the lanes
// that own keys of step j put their chunks where the scratch image wants them - chunk (key r,
// columns 16*ks + 8*h) belongs to fragment (dt = ks/2, u = (r/8)%2), slot pair
// 16*((r/4)%2) + 8*(ks%2) + 2*(r%4) + h - and the transposing reads hand them back as A
// fragments (cf. pv_from_scratch, which takes the rows in image order from global memory).
__device__ inline void pv_from_fragments(const Ctx &X, const uintx4 (&frag)[8], int j, bf16x8 pfj, floatx16 (&o)[4])
{
    if ((X.c32 >> 4) == j) {
        const int u = (X.c32 >> 3) & 1;
        lds_u8 *dst = X.scr + u * 512 + (16 * ((X.c32 >> 2) & 1) + 2 * (X.c32 & 3) + X.h) * 16;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
            *(lds_u128 *)(dst + (ks >> 1) * 1024 + (ks & 1) * 128) = frag[ks];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    bf16x8 va[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
        short4v lo = lds_read_tr(X.scr + X.lane * 8 + (dt * 2 + 0) * 512);
        short4v hi = lds_read_tr(X.scr + X.lane * 8 + (dt * 2 + 1) * 512);
        short8v v8 = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        __builtin_memcpy(&va[dt], &v8, 16);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[dt], pfj, o[dt], 0, 0, 0);
}

__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void bwd_dq_mfma_kernel(BwdArgs g, int npasses)
{
    const Args &a = g.f;
    extern __shared__ __align__(256) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X;
    X.lane = tid & 63;
    X.h = X.lane >> 5;
    X.c32 = X.lane & 31;
    X.Mtot = a.C * a.S * a.G;
    X.c = a.scale * kLog2e;
    X.k_lane = smem + X.lane * 16;                  // K row-major image of slot 0
    X.v_lane = smem + 2 * kTileBytes + X.lane * 8;  // K transposing image of slot 0
    X.scr = smem + 2 * kBwdSlotBytes + wave * kScrBytes;
    X.sv_row_lo = 4 * ((X.c32 >> 4) & 1) + ((X.c32 >> 1) & 3);
    X.sv_chunk_lo = 2 * ((X.c32 >> 3) & 1) + (X.c32 & 1);
    lds_u8 *vk_lane = smem + kTileBytes + X.lane * 16; // V row-major image of slot 0
    const int nblocks = (X.Mtot + kBlockRows - 1) / kBlockRows;
    const TileSlot t = make_tile_slot(tid);
    const int VH = a.Np * a.Hkv;
    // the gradient goes out through the forward pass's store routine: dq is laid out like q
    Args ad = a;
    ad.out = g.dq;
    ad.lse = nullptr;
    ad.o_sb = a.q_sb;
    ad.o_ss = a.q_ss;
    ad.o_sh = a.q_sh;

    for (int p = blockIdx.x; p < npasses; p += gridDim.x) {
        set_vhead(a, X, p % VH);
        const int blk_raw = (p / VH) * kNW + wave;
        const bool active = blk_raw < nblocks;
        const int blk = active ? blk_raw : nblocks - 1;
        const int r0 = blk * kBlockRows;
        const int ntiles = (X.P + kTileKeys - 1) / kTileKeys;
        const Row row = decode_row(a, X, blk);
        const bool rvalid = active && row.rin && (int)row.ri < clamp_len(a, row.rlen);
        const bool work = __builtin_amdgcn_ballot_w64(rvalid) != 0;

        // requested first, so that it is there with the rows below and costs no round trip of its own
        const float lse2 = (row.rin ? a.lse[((long long)row.rb * a.Hq + row.rh) * a.S + row.ri] : 0.f) * kLog2e;
        // Rows past their candidate's length take the data of its last position (never fetched
        // otherwise): what they compute is finite and stored as zero.
        Row rld = row;
        {
            const int len = clamp_len(a, row.rlen);
            rld.ri = (int)row.ri < len ? row.ri : (len > 0 ? (unsigned)(len - 1) : 0u);
        }
        uintx4 q[8], dof[8];
        load_q(a, X, rld, q);
        load_o_like(a, X, rld, g.dout, dof);
        float drow; // <dout_row, out_row>
        {
            uintx4 of[8];
            load_o_like(a, X, rld, a.out, of);
            drow = dout_dot_out(dof, of);
        }
        if (g.delta && rvalid && X.h == 0) // kept in the order of the stacked rows: see delta_index
            g.delta[delta_index(a, row.rb, row.rh, row.ri)] = drow;

        floatx16 o[4];
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                o[dt][e] = 0.f;

        // ---- prefix part: every row sees every prefix key ----
        if (ntiles > 0) {
            uintx4 kk, vk, kt2;
            auto fetch = [&](int kt) {
                uintx4 unused;
                load_tile_chunks(a, X, t, kt, kk, unused);   // K chunk for the row-major image; (V chunk of the transposing slot unused)
                // V chunk for the row-major image and K chunk for the transposing image
                const int last = X.P > 0 ? X.P - 1 : 0;
                const int kkey = kt * kTileKeys + t.k_row, vkey = kt * kTileKeys + t.v_row;
                vk = ld_global16(X.vpg + (long long)(kkey < X.P ? kkey : last) * a.kp_sp + t.k_chunk * 8);
                kt2 = ld_global16(X.kpg + (long long)(vkey < X.P ? vkey : last) * a.kp_sp + t.v_chunk * 8);
            };
            auto put = [&](int kt, int slot) {
                const int kkey = kt * kTileKeys + t.k_row, vkey = kt * kTileKeys + t.v_row;
                lds_u8 *s0 = smem + slot * kBwdSlotBytes + tid * 16;
                *(lds_u128 *)s0 = kkey < X.P ? kk : uintx4{0, 0, 0, 0};
                *(lds_u128 *)(s0 + kTileBytes) = kkey < X.P ? vk : uintx4{0, 0, 0, 0};
                *(lds_u128 *)(s0 + 2 * kTileBytes) = vkey < X.P ? kt2 : uintx4{0, 0, 0, 0};
            };
            fetch(0);
            __syncthreads(); // whatever the slots held has been used by every wavefront
            put(0, 0);
            __syncthreads();
            for (int kt = 0; kt < ntiles; ++kt) {
                fetch(kt + 1 < ntiles ? kt + 1 : kt);
                if (work) {
                    const int so = (kt & 1) * kBwdSlotBytes;
                    floatx16 s, dp;
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        s[e] = 0.f;
                        dp[e] = 0.f;
                    }
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks) {
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*(lds_u128 *)(X.k_lane + so + ks * 1024)),
                                                                    as_bf16x8(q[ks]), s, 0, 0, 0);
                        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(*(lds_u128 *)(vk_lane + so + ks * 1024)),
                                                                     as_bf16x8(dof[ks]), dp, 0, 0, 0);
                    }
                    const int nv = X.P - kt * kTileKeys - 4 * X.h; // element e holds key 8*(e/4) + e%4 + 4*h of the tile
                    bf16x8 pf[2];
                    if ((kt + 1) * kTileKeys <= X.P) // a full tile: every row sees all of it
                        ds_tile(s, dp, X.c, lse2, drow, [](int) { return true; }, pf);
                    else
                        ds_tile(s, dp, X.c, lse2, drow, [&](int e) { return 8 * (e >> 2) + (e & 3) < nv; }, pf);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int dt = 0; dt < 4; ++dt)
                            o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_fragment(X.v_lane + so, dt, j), pf[j], o[dt], 0,
                                                                            0, 0);
                }
                if (kt + 1 < ntiles)
                    put(kt + 1, (kt + 1) & 1);
                __syncthreads();
            }
        }

        // ---- suffix part: (candidate, 32-key step) pairs, wave-uniform ----
        if (work) {
            Ctx Xs = X; // the suffix V rows are fetched as row-major fragments too: the K loader pointed at V
            Xs.ksg = X.vsg;
            const int last_row = r0 + kBlockRows - 1 < X.Mtot ? r0 + kBlockRows - 1 : X.Mtot - 1;
            const int tok_first = fdiv(r0, a.div_g), tok_last = fdiv(last_row, a.div_g);
            const int bl_last = fdiv(tok_last, a.div_s);
            for (int bl = fdiv(tok_first, a.div_s); bl <= bl_last; ++bl) {
                const int b = X.cand0 + bl;
                const int len = len_uniform(a, b);
                const int i_lo = tok_first - bl * a.S > 0 ? tok_first - bl * a.S : 0;
                const int i_hi = tok_last - bl * a.S < a.S - 1 ? tok_last - bl * a.S : a.S - 1;
                const int kmax = i_hi < len - 1 ? i_hi : len - 1;
                if (i_lo >= len)
                    continue;
                for (int k0 = 0; k0 <= kmax; k0 += kTileKeys) {
                    floatx16 s, dp;
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        s[e] = 0.f;
                        dp[e] = 0.f;
                    }
                    // K rows once, as row-major fragments: A operands of S^T here, and the source of the
                    // transposed fragments of dQ^T further down
                    uintx4 kf[8];
                    load_suffix_k(a, X, b, k0, kmax, kf);
#pragma unroll
                    for (int ks = 0; ks < 8; ++ks)
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks]), as_bf16x8(q[ks]), s, 0, 0, 0);
                    {
                        uintx4 vf[8];
                        load_suffix_k(a, Xs, b, k0, kmax, vf); // V rows as row-major fragments
#pragma unroll
                        for (int ks = 0; ks < 8; ++ks)
                            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vf[ks]), as_bf16x8(dof[ks]), dp, 0, 0, 0);
                    }
                    // the row sees keys 0..ri of its own candidate; element e holds key k0 + 8*(e/4) + e%4 + 4*h
                    const int lim = ((int)row.rb == b ? (int)row.ri : -1) - k0 - 4 * X.h;
                    bf16x8 pf[2];
                    ds_tile(s, dp, X.c, lse2, drow, [&](int e) { return 8 * (e >> 2) + (e & 3) <= lim; }, pf);
                    pv_from_fragments(X, kf, 0, pf[0], o);
                    pv_from_fragments(X, kf, 1, pf[1], o);
                }
            }
        }
        if (active) {
            if (work) // store_block divides by the sum of both half-waves' l: 1/(2 * 0.5/scale) = scale
                store_block(ad, X, r0, row, rvalid, 0.f, 0.5f / a.scale, o);
            else
                store_zero_block(ad, X, r0, row);
        }
    }
}

// dq kernels work on 32-row blocks of one candidate: rows r0 .. r0+31 of its S*G stacked rows (i, g) of one KV
// head, the last block of a candidate being what is left.  Everything that depends on the candidate is
// then the same for all lanes, and a row's place within it fits 32 bits (block_offsets_fit).
struct DqBlock {
    int b, head;   // candidate and KV head
    int len;       // the candidate's clamped suffix length
    int r0;        // first row
    int i_lo, i_hi; // positions of the block's first and last existing row
    int ri, rh;    // this lane's row (rows past the candidate's last: that one)
    bool rvalid;   // ... exists and is not padding
};
__device__ inline DqBlock dq_block(const Args &a, const Ctx &X, int b, int head, int r0)
{
    DqBlock x;
    const int last = a.S * a.G - 1;
    x.b = b;
    x.head = head;
    x.len = len_uniform(a, b);
    x.r0 = r0;
    x.i_lo = (int)fdiv((unsigned)(r0 < last ? r0 : last), a.div_g);
    x.i_hi = (int)fdiv((unsigned)(r0 + kBlockRows - 1 < last ? r0 + kBlockRows - 1 : last), a.div_g);
    const int r = r0 + X.c32, rc = r < last ? r : last;
    x.ri = (int)fdiv((unsigned)rc, a.div_g);
    x.rh = head * a.G + rc - x.ri * a.G;
    x.rvalid = r <= last && x.ri < x.len;
    return x;
}

// Stores the block, or zeros.  This lane stores rows 8u + lane/8, 16 bytes at column 8*(lane%8) of either half.  (The
// row is decoded anew from a lane id that the compiler cannot trace back: no addresses held across the block.)
__device__ inline void store_dq(const BwdArgs &g, const Ctx &X, const DqBlock &x, bool zero, const floatx16 (&o)[4])
{
    const Args &a = g.f;
    int c = X.lane & 31;
    asm volatile("" : "+v"(c));
    const int last = a.S * a.G - 1;
    const int rs = x.r0 + c < last ? x.r0 + c : last;
    const int is = (int)fdiv((unsigned)rs, a.div_g);
    const unsigned off = ((unsigned)is * (unsigned)a.q_ss + (unsigned)(x.head * a.G + rs - is * a.G) * (unsigned)a.q_sh) * 2u;
    unsigned char *base = reinterpret_cast<unsigned char *>(g.dq) + (long long)x.b * a.q_sb * 2;
    unsigned short *dst[4];
    bool dst_ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int rl = 8 * u + (X.lane >> 3);
        dst[u] = reinterpret_cast<unsigned short *>(base + ((unsigned)__shfl((int)off, rl, 64) + 16u * (X.lane & 7)));
        dst_ok[u] = x.r0 + rl <= last;
        if (zero && dst_ok[u]) {
            __builtin_nontemporal_store(uintx4{0, 0, 0, 0}, reinterpret_cast<uintx4 *>(dst[u]));
            __builtin_nontemporal_store(uintx4{0, 0, 0, 0}, reinterpret_cast<uintx4 *>(dst[u] + 64));
        }
    }
    if (!zero)
        store_rows(X, dst, dst_ok, x.rvalid, a.scale, o);
}

// The rows of a block of one candidate from a tensor with the given row offsets (my_off: bytes from base
// to the row of lane c32), 8 rows x 128 bytes per request: register 4*half + g holds 16 bytes of row
// 8g + lane/8, chunk lane%8 of that half's columns.
__device__ inline void load_rows_block(const Ctx &X, const unsigned char *base, unsigned my_off, uintx4 (&raw)[2][4])
{
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
        const unsigned off = (unsigned)__shfl((int)my_off, 8 * g4 + (X.lane >> 3), 64) + 16u * (X.lane & 7);
        raw[0][g4] = *reinterpret_cast<const uintx4 *>(base + off);
        raw[1][g4] = *reinterpret_cast<const uintx4 *>(base + (off + 128u));
    }
}

// Suffix rows k0 .. k0+31 (base: row 0 of the candidate's K or V for this KV head; rows past kmax clamped: never visible).
__device__ inline void load_suffix_rows(const Args &a, const Ctx &X, const unsigned char *base, int k0, int kmax, uintx4 (&raw)[2][4])
{
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
        const int key = k0 + 8 * g4 + (X.lane >> 3);
        const unsigned off = (unsigned)(key < kmax ? key : kmax) * (unsigned)a.ks_ss * 2u + 16u * (X.lane & 7);
        raw[0][g4] = *reinterpret_cast<const uintx4 *>(base + off);
        raw[1][g4] = *reinterpret_cast<const uintx4 *>(base + (off + 128u));
    }
}

// Rows as they come turned into row-major fragments through the wavefront's scratch.
__device__ inline void rows_to_fragments(const Ctx &X, const HalfPlaces &hp, const uintx4 (&raw)[2][4], uintx4 (&f)[8])
{
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        half_put(hp, X.scr, raw[half]);
        scratch_fence();
#pragma unroll
        for (int i = 0; i < 4; ++i)
            f[4 * half + i] = half_row_frag(hp, X.scr, i);
        scratch_fence();
    }
}

// <dout_row, out_row> of the lane's row (c32) from rows as they come.
__device__ inline float rows_dot(const Ctx &X, const uintx4 (&x)[2][4], const uintx4 (&y)[2][4])
{
    float p[4];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4)
        p[g4] = sum8(chunk_dot(x[0][g4], y[0][g4])) + sum8(chunk_dot(x[1][g4], y[1][g4]));
    const float mine = X.lane & 2 ? (X.lane & 1 ? p[3] : p[2]) : (X.lane & 1 ? p[1] : p[0]); // row 8*(lane%4) + lane/8
    return __shfl(mine, 8 * (X.c32 & 7) + (X.c32 >> 3), 64);
}

// q and dout of the block as row-major fragments, and <dout_row, out_row> of the lane's row, left in the workspace
// as well.  Rows past the candidate's length take the data of its last position (what is padding is never fetched).
// between(): requests to be in flight together with these.
template <typename F>
__device__ inline float load_dq_block(const BwdArgs &g, const Ctx &X, const HalfPlaces &hp, const DqBlock &x, uintx4 (&q)[8],
                                      uintx4 (&dof)[8], F between)
{
    const Args &a = g.f;
    const int rld = x.ri < x.len ? x.ri : x.len - 1;
    const unsigned q_off = ((unsigned)rld * (unsigned)a.q_ss + (unsigned)x.rh * (unsigned)a.q_sh) * 2u;
    const unsigned o_off = ((unsigned)rld * (unsigned)a.o_ss + (unsigned)x.rh * (unsigned)a.o_sh) * 2u;
    const long long obase = (long long)x.b * a.o_sb * 2;
    uintx4 qr[2][4], dor[2][4], our[2][4];
    load_rows_block(X, reinterpret_cast<const unsigned char *>(a.q) + (long long)x.b * a.q_sb * 2, q_off, qr);
    load_rows_block(X, reinterpret_cast<const unsigned char *>(g.dout) + obase, o_off, dor);
    load_rows_block(X, reinterpret_cast<const unsigned char *>(a.out) + obase, o_off, our);
    between();
    rows_to_fragments(X, hp, qr, q);
    rows_to_fragments(X, hp, dor, dof);
    const float drow = rows_dot(X, dor, our);
    if (g.delta && x.rvalid && X.h == 0)
        g.delta[delta_index(a, x.b, x.rh, x.ri)] = drow;
    return drow;
}

// One 32-key tile whose K and V images (two half images each) are in LDS: dQ^T += K^T dS^T.  MASK: element
// e of the scores is visible iff its key offset 8*(e/4) + e%4 is <= lim.  Fragments are read kAheadFr
// sub-steps before their use, and nothing is moved across a sub-step: left to itself the compiler
// reads each one right before the matrix instruction that waits for it.
template <bool MASK>
__device__ __attribute__((always_inline)) void dq_tile(const HalfPlaces &hp, lds_u8 *kimg, lds_u8 *vimg, const uintx4 (&q)[8],
                                                       const uintx4 (&dof)[8], float c, float lse2, float drow, int lim,
                                                       floatx16 (&o)[4])
{
    constexpr int kAheadFr = 2;
    floatx16 s, dp;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        s[e] = 0.f;
        dp[e] = 0.f;
    }
    uintx4 kf[8], vf[8];
    bf16x8 kt[8]; // [4*j + dt]
    auto read = [&](int ks) {
        kf[ks] = half_row_frag(hp, kimg + (ks >> 2) * kHalfBytes, ks & 3);
        vf[ks] = half_row_frag(hp, vimg + (ks >> 2) * kHalfBytes, ks & 3);
    };
    auto read_t = [&](int i) { kt[i] = half_col_frag(hp, kimg + ((i & 3) >> 1) * kHalfBytes, i & 1, i >> 2); };
#pragma unroll
    for (int i = 0; i < kAheadFr; ++i)
        read(i);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        if (ks + kAheadFr < 8)
            read(ks + kAheadFr);
        else {
            read_t(2 * (ks + kAheadFr - 8));
            read_t(2 * (ks + kAheadFr - 8) + 1);
        }
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kf[ks]), as_bf16x8(q[ks]), s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vf[ks]), as_bf16x8(dof[ks]), dp, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
    bf16x8 pf[2];
    if constexpr (MASK)
        ds_tile(s, dp, c, lse2, drow, [&](int e) { return 8 * (e >> 2) + (e & 3) <= lim; }, pf);
    else
        ds_tile(s, dp, c, lse2, drow, [](int) { return true; }, pf);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (i + 4 < 8)
            read_t(i + 4);
        o[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[i], pf[i >> 2], o[i & 3], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// ------------------------------------------------------------------------------------------
// dq with the prefix resident in LDS (prefix of at most 256 rows).  A persistent workgroup copies
// the prefix K and V of its (instruction, KV head) pair into LDS once; its eight wavefronts
// then walk independently, without any further workgroup barrier, over the pair's blocks, each inside one candidate.
// One image per 32-key tile and tensor serves all three products: V is read row-major for
// dP^T = V dO^T, K row-major for S^T = K Q^T and transposed for K^T dS^T.
//
// What bounds it: matrix instructions (half of a SIMD's time at P = 256), then the LDS and vector work of a
// block's start, which two wavefronts per SIMD - the registers allow no third - hide in part.  1024 candidates of
// 16..24 positions x 4 heads, 8 KV heads, P 256: 195 us (208 us with rows fetched as fragments, 32 bytes of 32 rows
// at a time, the own keys last, and fragments read where the compiler put the reads); a plain copy of its
// bytes takes 128 us.
// ------------------------------------------------------------------------------------------
constexpr int kDqMaxTiles = 8;

__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void bwd_dq_resident_kernel(BwdArgs g, int nb, FastDiv div_nb, int per_vh, int vh_slots, int max_tiles)
{
    const Args &a = g.f;
    extern __shared__ __align__(256) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X;
    X.lane = tid & 63;
    X.h = X.lane >> 5;
    X.c32 = X.lane & 31;
    X.c = a.scale * kLog2e;
    X.scr = smem + 2 * max_tiles * kTileBytes + wave * kScrBytes;
    const HalfPlaces hp = half_places(X.lane);
    const int nblocks = a.C * nb;
    const int blk_stride = per_vh * kNW;
    const int VH = a.Np * a.Hkv;
    for (int vh = blockIdx.x % vh_slots; vh < VH; vh += vh_slots) {
        set_vhead(a, X, vh);
        const int T = (X.P + kTileKeys - 1) / kTileKeys;
        __syncthreads(); // every wavefront is done with the images of the virtual head before
        { // Each wavefront copies one half image (K or V, 64 columns) of every other tile, two of them at a time.
            // Rows past the prefix: its last row stands in (never visible).
            const int last = X.P > 0 ? X.P - 1 : 0, which = wave & 3;
            const unsigned short *src = (which < 2 ? X.kpg : X.vpg) + 64 * (which & 1) + 8 * (X.lane & 7);
            for (int kt0 = wave >> 2; kt0 < T; kt0 += 4) {
                uintx4 st[2][4] = {};
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (kt0 + 2 * i < T)
#pragma unroll
                        for (int g4 = 0; g4 < 4; ++g4) {
                            const int key = (kt0 + 2 * i) * kTileKeys + 8 * g4 + (X.lane >> 3);
                            st[i][g4] = ld_global16(src + (long long)(key < X.P ? key : last) * a.kp_sp);
                        }
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    if (kt0 + 2 * i < T)
                        half_put(hp, smem + (kt0 + 2 * i) * 2 * kTileBytes + which * kHalfBytes, st[i]);
            }
        }
        __syncthreads();

        for (int blk = (blockIdx.x / vh_slots) * kNW + wave; blk < nblocks; blk += blk_stride) {
            const int bl = __builtin_amdgcn_readfirstlane((int)fdiv((unsigned)blk, div_nb));
            const DqBlock row = dq_block(a, X, X.cand0 + bl, X.head, (blk - bl * nb) * kBlockRows);
            floatx16 o[4];
            if (row.i_lo >= row.len) { // nothing but padding
                store_dq(g, X, row, true, o);
                continue;
            }
            const int kmax = row.i_hi < row.len - 1 ? row.i_hi : row.len - 1;

            // requested first, so that it is there with the rows below and costs no round trip of its own
            const float lse2 = a.lse[((long long)row.b * a.Hq + row.rh) * a.S + row.ri] * kLog2e;
            uintx4 q[8], dof[8], kr[2][4], vr[2][4];
            const unsigned char *ksb = reinterpret_cast<const unsigned char *>(X.ksg) + (long long)row.b * a.ks_sb * 2;
            const unsigned char *vsb = reinterpret_cast<const unsigned char *>(X.vsg) + (long long)row.b * a.ks_sb * 2;
            const float drow = load_dq_block(g, X, hp, row, q, dof, [&] { // <dout_row, out_row>
                load_suffix_rows(a, X, ksb, 0, kmax, kr);
                load_suffix_rows(a, X, vsb, 0, kmax, vr);
            });

            // ---- suffix part: 32-key steps of the block's own candidate ----
            auto suffix_step = [&](int k0, auto first) {
                floatx16 s, dp;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    s[e] = 0.f;
                    dp[e] = 0.f;
                }
                bf16x8 kt[2][4]; // K^T fragments
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    half_put(hp, X.scr, kr[half]);
                    scratch_fence();
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(half_row_frag(hp, X.scr, i)), as_bf16x8(q[4 * half + i]), s, 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int d = 0; d < 2; ++d)
                            kt[j][2 * half + d] = half_col_frag(hp, X.scr, d, j);
                    scratch_fence();
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    half_put(hp, X.scr, vr[half]);
                    scratch_fence();
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(half_row_frag(hp, X.scr, i)), as_bf16x8(dof[4 * half + i]), dp, 0, 0, 0);
                    scratch_fence();
                    __builtin_amdgcn_sched_barrier(0);
                }
                // the row sees keys 0..ri of its candidate; element e holds key k0 + 8*(e/4) + e%4 + 4*h
                const int lim = row.ri - k0 - 4 * X.h;
                bf16x8 pf[2];
                ds_tile(s, dp, X.c, lse2, drow, [&](int e) { return 8 * (e >> 2) + (e & 3) <= lim; }, pf);
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) {
                        if (decltype(first)::value && j == 0)
#pragma unroll
                            for (int e = 0; e < 16; ++e)
                                o[dt][e] = 0.f;
                        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[j][dt], pf[j], o[dt], 0, 0, 0);
                    }
            };
            suffix_step(0, std::true_type{});
            for (int k0 = kTileKeys; k0 <= kmax; k0 += kTileKeys) {
                load_suffix_rows(a, X, ksb, k0, kmax, kr);
                load_suffix_rows(a, X, vsb, k0, kmax, vr);
                suffix_step(k0, std::false_type{});
            }

            // ---- prefix part: every row sees every prefix key (only a ragged last tile has keys to hide) ----
            int kt = 0;
            for (; kt < X.P / kTileKeys; ++kt) {
                lds_u8 *img = smem + kt * 2 * kTileBytes;
                dq_tile<false>(hp, img, img + kTileBytes, q, dof, X.c, lse2, drow, 0, o);
            }
            if (kt < T) {
                lds_u8 *img = smem + kt * 2 * kTileBytes;
                dq_tile<true>(hp, img, img + kTileBytes, q, dof, X.c, lse2, drow, X.P - 1 - kt * kTileKeys - 4 * X.h, o);
            }

            store_dq(g, X, row, false, o);
        }
    }
}

// ------------------------------------------------------------------------------------------
// The same over packed rows (pskv_packed.hpp): calls with suffix lengths, S <= 64.  A block's own keys are its window's.
// Bound as the kernel above; it has fewer blocks (20480 for 23700 at the size named there: the whole backward pass 299 -> 281 us),
// ranges of blocks that differ by one at most (or blocks in turn), and its prefix straight into LDS.  Ranges next to each other belong to different
// workgroups: handing a workgroup eight neighbouring ones cost 2 % over 74 calls, 7 % where a wavefront has a few blocks.
// ------------------------------------------------------------------------------------------
struct DqPacked {
    BwdArgs g;
    PackedArgs pa;
    int per_vh, vh_slots, max_tiles;
};

template <int STEPS>
__global__ __attribute__((amdgpu_flat_work_group_size(512, 512), amdgpu_waves_per_eu(2, 2)))
void bwd_dq_packed_kernel(DqPacked call)
{
    extern __shared__ __align__(256) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int VH = call.g.f.Np * call.g.f.Hkv, slots = call.vh_slots;
    for (int vh = __builtin_amdgcn_readfirstlane(blockIdx.x % slots); vh < VH; vh += slots) {
        const DqPacked &call = first_parameter<DqPacked>(); // (read again, as in the forward kernel)
        const BwdArgs &g = call.g;
        const Args &a = g.f;
        const PackedArgs &pa = call.pa;
        const int per_vh = call.per_vh, max_tiles = call.max_tiles;
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        Ctx X;
        X.lane = tid & 63;
        X.h = X.lane >> 5;
        X.c32 = X.lane & 31;
        X.c = a.scale * kLog2e;
        X.scr = smem + 2 * max_tiles * kTileBytes + wave * kScrBytes;
        const HalfPlaces hp = half_places(X.lane);
        const int slice = __builtin_amdgcn_readfirstlane(blockIdx.x / call.vh_slots), per_chunk = (a.C + kLenChunks - 1) / kLenChunks;
        const int waves = per_vh * kNW, me = wave * per_vh + slice;
        lds_int *const lens = (lds_int *)(smem + 2 * max_tiles * kTileBytes); // (in the scratch)
        set_vhead(a, X, vh);
        const int T = (X.P + kTileKeys - 1) / kTileKeys;
        __syncthreads(); // every wavefront is done with the images and the scratch of the virtual head before
        int fresh = tid; // (what is worked out from it is not kept over the block loop)
        asm volatile("" : "+v"(fresh));
        if (wave < kLenWaves) { // four wavefronts add the lengths up ...
            ChunkRows mine = {0, 0};
            for (int k0 = 0; k0 < per_chunk; k0 += kLenRound) {
                int len[kLenRound];
                const int n = per_chunk - k0 < kLenRound ? per_chunk - k0 : kLenRound;
                load_lengths(a, X.cand0, per_chunk, k0, n, fresh, len);
                count_lengths(a, per_chunk, k0, n, len, lens, fresh, mine);
            }
            add_up(mine, lens, fresh);
        } else { // ... and each of the others requests one half image (K or V, 64 columns) of every tile, straight into LDS:
                 // lane l's bytes go to slot l/8 and place l%8 of a piece of eight rows (see HalfPlaces).
                 // Rows past the prefix: its last row stands in (never visible).
            const int which = wave & 3, slot = (fresh & 63) >> 3, place = fresh & 7;
            const unsigned row = (unsigned)a.kp_sp * 2u;
            const unsigned char *src = reinterpret_cast<const unsigned char *>(which < 2 ? X.kpg : X.vpg) + 128 * (which & 1);
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const int k = slot ^ (g4 & 1), left = X.P - t * kTileKeys - 1, r = 8 * g4 + k;
                    request_to_lds(src + (unsigned)(t * kTileKeys) * row, (unsigned)(r < left ? r : left) * row + ((place ^ half_swz(k)) << 4),
                                   smem + t * 2 * kTileBytes + which * kHalfBytes + g4 * 1024);
                }
        }
        __syncthreads();
        const PackedList list = choose_list<STEPS>(a, pa, T, waves, per_chunk, lens);
        const int nblocks = (list.total + kBlockRows - 1) / kBlockRows;
        const int each = (int)fdiv(nblocks, pa.div_w), over = nblocks - each * waves;
        int blk_lo = me * each + (me < over ? me : over), blk_hi = blk_lo + each + (me < over ? 1 : 0), step = 1; // from blk_lo, every step-th
        // Blocks in turn where places are a division away and each key head has one query head, as in the forward kernel (us for the whole backward pass,
        // ranges and in turn, 32/32 heads, P 128: 64 x 28: 45.3, 42.5; 256 x 16..32: 136, 132; 700 x 32: 437, 432; before this kernel 43.9, 132, 432).
        if (list.even && list.align > 1 && a.G == 1) {
            step = waves;
            blk_lo = slice * kNW + wave;
            blk_hi = nblocks;
        }
        Walk w = {X.cand0, 0, 0};
        if (blk_lo < blk_hi)
            w = find_row(a, list, X.cand0, blk_lo * kBlockRows, fresh & 63);
        PSKV_WAIT_VM(0);
        asm volatile("" ::: "memory");
        __syncthreads();

        const int row_hi = blk_hi * kBlockRows < list.total ? blk_hi * kBlockRows : list.total;
        int pad = me;
        for (int r0 = blk_lo * kBlockRows; r0 < row_hi;) {
            unsigned q_off;
            PackedRow row;
            if (step > 1) {
                w = walk_even(a, pa.div_run, kBlockRows, r0);
                w.b += X.cand0;
                w.len = packed_len(a, w.b);
            }
            const PackedBlock<STEPS> x = packed_block<STEPS>(a, pa, fresh_lane(X), w, r0, list, q_off, row);
            const int next = step > 1 ? step * kBlockRows : x.rows; // (a block of 32 rows, or of fewer where the next candidate is far away)
            r0 = row_hi - r0 > next ? r0 + next : row_hi;           // (the sum may need more than 32 bits)
            const int rh = X.head * a.G + row.gq, b = x.b + (int)(row.from >> 6), ri = (int)(row.from & 63);

            // requested first, so that it is there with the rows below and costs no round trip of its own
            const float lse2 = a.lse[((long long)b * a.Hq + rh) * a.S + ri] * kLog2e;
            uintx4 q[8], dof[8], kr[2][4], vr[2][4];
            const unsigned char *ksb = reinterpret_cast<const unsigned char *>(X.ksg) + (unsigned long long)(unsigned)x.b * pa.k_sb;
            const unsigned char *vsb = reinterpret_cast<const unsigned char *>(X.vsg) + (unsigned long long)(unsigned)x.b * pa.k_sb;
            auto window_rows = [&](int k0) __attribute__((always_inline)) { // the window's rows k0 .. k0 + 31, eight per request
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const unsigned e = window_entry(x, k0 + 8 * g4 + (X.lane >> 3));
                    const unsigned off = packed_off(e, pa.k_sb, pa.k_ss) + 16u * (X.lane & 7);
                    kr[0][g4] = *reinterpret_cast<const uintx4 *>(ksb + off);
                    kr[1][g4] = *reinterpret_cast<const uintx4 *>(ksb + (off + 128u));
                    vr[0][g4] = *reinterpret_cast<const uintx4 *>(vsb + off);
                    vr[1][g4] = *reinterpret_cast<const uintx4 *>(vsb + (off + 128u));
                }
            };
            float drow;
            {
                const unsigned o_off = packed_off(row.from, pa.o_sb, pa.o_ss) + __umul24(rh, pa.o_sh);
                const unsigned long long obase = (unsigned long long)(unsigned)x.b * pa.o_sb;
                uintx4 qr[2][4], dor[2][4], our[2][4];
                load_rows_block(X, reinterpret_cast<const unsigned char *>(a.q) + (unsigned long long)(unsigned)x.b * pa.q_sb, q_off, qr);
                load_rows_block(X, reinterpret_cast<const unsigned char *>(g.dout) + obase, o_off, dor);
                load_rows_block(X, reinterpret_cast<const unsigned char *>(a.out) + obase, o_off, our);
                window_rows(0);
                rows_to_fragments(X, hp, qr, q);
                rows_to_fragments(X, hp, dor, dof);
                drow = rows_dot(X, dor, our);
                if (g.delta && row.own == row.from && X.h == 0)
                    g.delta[delta_index(a, b, rh, ri)] = drow;
            }
            floatx16 o[4];
            // ---- the window ----
            auto window_step = [&](int k0, auto first) __attribute__((always_inline)) {
                floatx16 s, dp;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    s[e] = 0.f;
                    dp[e] = 0.f;
                }
                bf16x8 kt[2][4]; // K^T fragments
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    half_put(hp, X.scr, kr[half]);
                    scratch_fence();
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(half_row_frag(hp, X.scr, i)), as_bf16x8(q[4 * half + i]), s, 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int d = 0; d < 2; ++d)
                            kt[j][2 * half + d] = half_col_frag(hp, X.scr, d, j);
                    scratch_fence();
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    half_put(hp, X.scr, vr[half]);
                    scratch_fence();
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(half_row_frag(hp, X.scr, i)), as_bf16x8(dof[4 * half + i]), dp, 0, 0, 0);
                    scratch_fence();
                    __builtin_amdgcn_sched_barrier(0);
                }
                const int bits = sees_bits(x, k0, X.h);
                bf16x8 pf[2];
                ds_tile(s, dp, X.c, lse2, drow, [&](int e) { return (bits >> (8 * (e >> 2) + (e & 3)) & 1) != 0; }, pf);
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) {
                        if (decltype(first)::value && j == 0)
#pragma unroll
                            for (int e = 0; e < 16; ++e)
                                o[dt][e] = 0.f;
                        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt[j][dt], pf[j], o[dt], 0, 0, 0);
                    }
            };
            window_step(0, std::true_type{});
            if (STEPS > 1 && x.width > kTileKeys) {
                window_rows(kTileKeys);
                window_step(kTileKeys, std::false_type{});
            }

            // ---- prefix part: every row sees every prefix key (only a ragged last tile has keys to hide) ----
            int kt = 0;
            for (; kt < X.P / kTileKeys; ++kt) {
                lds_u8 *img = smem + kt * 2 * kTileBytes;
                dq_tile<false>(hp, img, img + kTileBytes, q, dof, X.c, lse2, drow, 0, o);
            }
            if (kt < T) {
                lds_u8 *img = smem + kt * 2 * kTileBytes;
                dq_tile<true>(hp, img, img + kTileBytes, q, dof, X.c, lse2, drow, X.P - 1 - kt * kTileKeys - 4 * X.h, o);
            }

            { // (the row is found anew: no addresses held across the block)
                const Ctx Y = fresh_lane(X);
                const PackedRow y = packed_row(a, x, Y.c32, list.align);
                const unsigned off = packed_off(y.own, pa.q_sb, pa.q_ss) + __umul24(Y.head * a.G + y.gq, pa.q_sh);
                const int rows = list.align > 1 ? a.S * a.G - (x.r0 - x.first) : x.rows; // that exist
                unsigned char *base = reinterpret_cast<unsigned char *>(g.dq) + (unsigned long long)(unsigned)x.b * pa.q_sb;
                unsigned short *dst[4];
                bool dst_ok[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int rl = 8 * u + (Y.lane >> 3);
                    dst[u] = reinterpret_cast<unsigned short *>(base + ((unsigned)__shfl((int)off, rl, 64) + 16u * (Y.lane & 7)));
                    dst_ok[u] = rl < rows;
                }
                store_rows(Y, dst, dst_ok, y.own == y.from, a.scale, o);
            }
            if (pad < a.C) {
                store_padding(a, fresh_lane(X), X.cand0 + pad, packed_len(a, X.cand0 + pad), list.align, g.dq, pa.q_sb, pa.q_ss, pa.q_sh, nullptr);
                pad += waves;
            }
        }
        for (; pad < a.C; pad += waves)
            store_padding(a, fresh_lane(X), X.cand0 + pad, packed_len(a, X.cand0 + pad), list.align, g.dq, pa.q_sb, pa.q_ss, pa.q_sh, nullptr);
    }
}

// ------------------------------------------------------------------------------------------
// dq with prefix and own keys shared in LDS.  A pass is four 32-row blocks of one (candidate, KV head) unit, one
// per wavefront; the prefix tiles and then the candidate's own keys, as far as any of the four blocks sees them,
// go through two LDS slots, one barrier per tile, the next tile's rows on their way meanwhile.  The causal
// order makes the four blocks of a pass need nearly the same own tiles.  Two such workgroups share a compute
// unit, so that one works while the other one waits at its barrier or for the rows of its next pass.
//
// What bounds it: the start of a pass (rows of q, dout and out from HBM, their change into fragments and
// <dout,out>: 7 of 30 thousand cycles), the tiles' matrix instructions (1500 cycles per tile and wavefront pair) and
// staging (900).  256 candidates of 128..160 positions x 4 heads, 8 KV heads, P 128: 330 us (376 us with the own keys fetched by
// each wavefront for itself, two round trips per 32 of them); a plain copy of its bytes takes 225 us.
// ------------------------------------------------------------------------------------------
constexpr int kUnitWaves = 4;
constexpr int kUnitLdsBytes = 2 * 2 * kTileBytes + kUnitWaves * kHalfBytes;

struct UnitShape {
    int npc; // passes per (candidate, KV head): groups of kUnitWaves 32-row blocks of its S*G rows
    FastDiv div_npc, div_hkv;
};

__global__ __attribute__((amdgpu_flat_work_group_size(kUnitWaves * 64, kUnitWaves * 64), amdgpu_waves_per_eu(2, 2)))
void bwd_dq_unit_kernel(BwdArgs g, UnitShape us, int npasses)
{
    const Args &a = g.f;
    extern __shared__ __align__(256) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Ctx X;
    X.lane = tid & 63;
    X.h = X.lane >> 5;
    X.c32 = X.lane & 31;
    X.c = a.scale * kLog2e;
    X.scr = smem + 4 * kTileBytes + wave * kHalfBytes;
    const HalfPlaces hp = half_places(X.lane);
    const int rows_c = a.S * a.G; // stacked rows of one candidate
    const int r8 = X.lane >> 3;
    // this wavefront stages one half image of every tile: K columns 0..63, 64..127, V columns 0..63, 64..127
    const int stage_off = wave * kHalfBytes, stage_col = 64 * (wave & 1) + 8 * (X.lane & 7);
    int slot = 0;

    for (int p = blockIdx.x; p < npasses; p += gridDim.x) {
        // pass ids: the passes of one unit are 8 apart - on one XCD -, the longest (last rows) first
        const int y = p >> 3;
        const int uy = (int)fdiv((unsigned)y, us.div_npc), pc = us.npc - 1 - (y - uy * us.npc);
        const int unit = uy * 8 + (p & 7);
        if (unit >= a.B * a.Hkv)
            continue; // (the same for the whole workgroup)
        const int b = (int)fdiv((unsigned)unit, us.div_hkv), head = unit - b * a.Hkv;
        const int n = a.Np > 1 ? b / a.C : 0;
        set_vhead(a, X, n * a.Hkv + head);
        const int T = (X.P + kTileKeys - 1) / kTileKeys;
        const int r_first = pc * (kUnitWaves * kBlockRows);
        const DqBlock row = dq_block(a, X, b, head, r_first + wave * kBlockRows);
        floatx16 o[4];
        if ((int)fdiv((unsigned)r_first, a.div_g) >= row.len) { // nothing but padding (the same for the whole workgroup)
            store_dq(g, X, row, true, o);
            continue;
        }
        const bool work = row.r0 < rows_c && row.i_lo < row.len;
        const int kmax_w = row.i_hi < row.len - 1 ? row.i_hi : row.len - 1; // last own key this wavefront's rows see
        const int r_last = r_first + kUnitWaves * kBlockRows - 1 < rows_c ? r_first + kUnitWaves * kBlockRows - 1 : rows_c - 1;
        const int i_hi_pass = (int)fdiv((unsigned)r_last, a.div_g);
        const int kmax = i_hi_pass < row.len - 1 ? i_hi_pass : row.len - 1;
        const int ntiles = T + kmax / kTileKeys + 1;

        const unsigned short *stage_pre = (wave < 2 ? X.kpg : X.vpg) + stage_col;
        const unsigned short *stage_own = (wave < 2 ? X.ksg : X.vsg) + (long long)b * a.ks_sb + stage_col;
        uintx4 st[4];
        auto fetch = [&](int t) {
            const bool own = t >= T;
            const unsigned short *base = own ? stage_own : stage_pre;
            const long long stride = own ? a.ks_ss : a.kp_sp;
            const int first = (own ? t - T : t) * kTileKeys + r8, last = own ? kmax : X.P - 1; // (rows past the last one are never visible)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int key = first + 8 * g4 < last ? first + 8 * g4 : last;
                st[g4] = ld_global16(base + (long long)key * stride);
            }
        };
        fetch(0);

        const float lse2 = a.lse[((long long)b * a.Hq + row.rh) * a.S + row.ri] * kLog2e;
        uintx4 q[8], dof[8];
        const float drow = load_dq_block(g, X, hp, row, q, dof, [] {}); // <dout_row, out_row>

#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                o[dt][e] = 0.f;

        // Tile t goes into its slot, tile t+1 is requested.
        auto stage = [&](int t) {
            lds_u8 *img = smem + slot * 2 * kTileBytes;
            half_put(hp, img + stage_off, st); // (its last readers are past the barrier of the tile before)
            __syncthreads();
            fetch(t + 1 < ntiles ? t + 1 : t);
            slot ^= 1;
            return img;
        };
        // Elements of the scores: key 8*(e/4) + e%4 + 4*h of the tile.  Whole prefix tiles, seen by every row; the
        // prefix's last, ragged one and the own keys as far as this wavefront's rows see any; what is left for others.
        const int nfull = work ? X.P / kTileKeys : 0, nmine = work ? T + kmax_w / kTileKeys + 1 : 0;
        int t = 0;
        for (; t < nfull; ++t) {
            lds_u8 *img = stage(t);
            dq_tile<false>(hp, img, img + kTileBytes, q, dof, X.c, lse2, drow, 0, o);
        }
        for (; t < nmine; ++t) {
            lds_u8 *img = stage(t);
            const int lim = (t < T ? X.P - 1 - t * kTileKeys : row.ri - (t - T) * kTileKeys) - 4 * X.h;
            dq_tile<true>(hp, img, img + kTileBytes, q, dof, X.c, lse2, drow, lim, o);
        }
        for (; t < ntiles; ++t)
            stage(t);
        store_dq(g, X, row, !work, o);
    }
}

// ------------------------------------------------------------------------------------------
// dk_suf, dv_suf on the matrix cores.  One workgroup of two wavefronts per (candidate, KV head, tile
// of 32 suffix keys); wavefront DH owns half DH of the 128 columns (the accumulators of both halves
// would not fit one register file).  The pair walks over the candidate's 32-row blocks of stacked
// query rows (i, g) that can see the tile and accumulates, in the non-transposed formulation (a lane
// owns one key column):
//     S   = Q K^T          A = Q fragment,   B = K fragment
//     dP  = dO V^T         A = dO fragment,  B = V fragment
//     P   = exp2(c S - lse),  dS = P o (dP - D)      per element: row quantities come through LDS
//     dV^T += dO^T P       A = dO^T fragment,  B = P packed to bf16
//     dK^T += Q^T dS       A = Q^T fragment,   B = dS packed to bf16
// The rows of q and dout go through half images in LDS, from which both kinds of fragments are read.
// The first two products contract over the 128 columns: each wavefront forms its own half of that
// sum from its own half of the columns of q, dout, K and V - the only columns it ever fetches, so
// that every row of q and dout crosses HBM once per tile and not once per wavefront - and the
// halves change hands through LDS: a wavefront completes S and dP, and takes the exponentials,
// for one of the block's two 16-row steps only (it receives the other wavefront's half of the
// sums for those rows, 2 KB each of S and dP in fp32) and passes that step's packed P and dS on
// to the other one.  The second products need exactly the columns the wavefront already holds.
// The accumulators of S hold, for lane half h, rows 8*kk + 4*h + t of the block in element
// 4*kk + t: exactly the order in which the transposed fragments hold the rows of dO and Q, so P
// and dS go from the first products to the second ones through registers only.
//
// What bounds it: the chain load - LDS - products - exchange - weights - exchange - products of a block, 4000 cycles
// with two wavefronts per SIMD, and at short suffixes HBM.  256 candidates of 128..160 positions x 4 heads, 8 KV
// heads: 221 us (258 us with rows fetched as fragments); stepping from block to block by additions matters
// as much as whole lines (offsets shuffled between the lanes: a block's requests took 1300..2500
// cycles to issue, now 400).
// ------------------------------------------------------------------------------------------
constexpr int kDkvWaves = 2; // the two column halves of one unit
constexpr int kDkvScrBytes = 2 * kHalfBytes; // per wavefront: images of dO and Q
constexpr int kDkvAux = 512; // per wavefront: lse, <dout,out> and suffix position of the block's 32 rows
constexpr int kDkvXchBytes = 2 * 8 * 256 + 2 * 1024; // per wavefront, for the other one: its halves of S and dP for that one's
                                                     // 16-row step (8 accumulator registers of 256 bytes each), then its own
                                                     // step's packed weights and score gradients
constexpr int kDkvLdsBytes = kDkvWaves * (kDkvScrBytes + kDkvAux + kDkvXchBytes) + 256; // + the halves of <dout,out>

template <int DH, bool HAS_DELTA, bool FIT>
__device__ __attribute__((always_inline)) void bwd_dkv_unit(const BwdArgs &g, lds_u8 *smem, int tid, int bk, int kt)
{
    const Args &a = g.f;
    const int k = bk % a.Hkv, b = bk / a.Hkv;
    const int k0 = kt * kTileKeys;

    Ctx X;
    X.lane = tid & 63;
    X.h = X.lane >> 5;
    X.c32 = X.lane & 31;
    X.Mtot = a.S * a.G; // rows of this candidate
    X.c = a.scale * kLog2e;
    X.scr = smem + DH * (kDkvScrBytes + kDkvAux);
    const HalfPlaces hp = half_places(X.lane);
    lds_u8 *img_o = X.scr, *img_q = X.scr + kHalfBytes; // the block's rows of dO and Q
    const int row8 = X.lane >> 3;                       // this lane fetches rows 8g + row8, chunk lane%8
    typedef __attribute__((address_space(3))) float lds_f32;
    typedef __attribute__((address_space(3))) floatx4 lds_f32x4;
    lds_f32 *aux_lse = (lds_f32 *)(X.scr + kDkvScrBytes);
    lds_f32 *aux_drow = aux_lse + 32;
    lds_f32 *aux_i = aux_drow + 32; // suffix position of the row as a float, -1 for a row that does not count
    // where the halves of S and dP change hands: mine to write, the other wavefront's to read
    lds_u8 *xch = smem + kDkvWaves * (kDkvScrBytes + kDkvAux);
    lds_u8 *xch_mine = xch + DH * kDkvXchBytes + X.lane * 16, *xch_other = xch + (1 - DH) * kDkvXchBytes + X.lane * 16;
    lds_f32 *xdrow = (lds_f32 *)(xch + kDkvWaves * kDkvXchBytes); // [2][32]: the halves of <dout,out>

    const int len = len_uniform(a, b);
    const int key = k0 + X.c32; // this lane's key
    floatx16 dk[2], dv[2]; // output columns 64*DH .. 64*DH+63
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            dk[dt][e] = 0.f;
            dv[dt][e] = 0.f;
        }

    if (k0 < len) { // the same for both wavefronts of the workgroup: the barriers below are met by both
        const int kmax = len - 1;
        const unsigned char *qb = reinterpret_cast<const unsigned char *>(a.q) + ((long long)b * a.q_sb + (long long)k * a.G * a.q_sh) * 2;
        const long long ob = ((long long)b * a.o_sb + (long long)k * a.G * a.o_sh) * 2;
        const unsigned char *dob = reinterpret_cast<const unsigned char *>(g.dout) + ob;
        const unsigned char *outb = reinterpret_cast<const unsigned char *>(a.out) + ob;
        const int nrows = len * a.G; // rows (i, g) with i < len, in stacked order i*G + g
        // this half's columns of the tile's K and V rows as row-major fragments (rows past kmax clamped:
        // never visible): the same for every block of rows
        uintx4 kfh[4], vfh[4];
        {
            const unsigned short *ksb = reinterpret_cast<const unsigned short *>(a.ks) + (long long)b * a.ks_sb + (long long)k * a.ks_sh;
            const unsigned short *vsb = reinterpret_cast<const unsigned short *>(a.vs) + (long long)b * a.ks_sb + (long long)k * a.ks_sh;
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int krow = k0 + 8 * g4 + row8 < kmax ? k0 + 8 * g4 + row8 : kmax;
                const long long koff = (long long)krow * a.ks_ss + 8 * (X.lane & 7) + 64 * DH;
                kfh[g4] = ld_global16(ksb + koff);
                vfh[g4] = ld_global16(vsb + koff);
            }
            half_put(hp, img_o, kfh);
            half_put(hp, img_q, vfh);
            scratch_fence();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                kfh[i] = half_row_frag(hp, img_o, i);
                vfh[i] = half_row_frag(hp, img_q, i);
            }
            scratch_fence();
        }
        // What a block needs from global memory, all requested in one round trip: this half's columns
        // of q and dout and the row quantities of this lane's row (c32) of the block.
        struct BlockIn {
            uintx4 qr[4], dor[4]; // as they come: rows 8g + row8
            float lse_row, drow;
        };
        // Where those rows are.  Row rl = i*G + g of the candidate; a block further down every row's g goes
        // down by 32 modulo G, and where that would be negative another position is borrowed: no divisions
        // and no products in the loop.
        typedef typename std::conditional<FIT, unsigned, long long>::type off_t; // bytes
        struct Place {
            off_t q, o; // rows of q and of dout and out
            int gq;
        };
        const off_t chunk_off = 16 * (X.lane & 7) + 128 * DH;
        auto place = [&](int rl, Place &x) {
            const int ri = (int)fdiv((unsigned)rl, a.div_g);
            x.gq = rl - ri * a.G;
            x.q = ((off_t)ri * (off_t)a.q_ss + (off_t)x.gq * (off_t)a.q_sh) * 2 + chunk_off;
            x.o = ((off_t)ri * (off_t)a.o_ss + (off_t)x.gq * (off_t)a.o_sh) * 2 + chunk_off;
        };
        const int step_i = (int)fdiv((unsigned)kBlockRows, a.div_g), step_g = kBlockRows - step_i * a.G;
        const off_t step_q = ((off_t)step_i * (off_t)a.q_ss + (off_t)step_g * (off_t)a.q_sh) * 2;
        const off_t step_o = ((off_t)step_i * (off_t)a.o_ss + (off_t)step_g * (off_t)a.o_sh) * 2;
        const off_t borrow_q = ((off_t)a.G * (off_t)a.q_sh - (off_t)a.q_ss) * 2, borrow_o = ((off_t)a.G * (off_t)a.o_sh - (off_t)a.o_ss) * 2;
        Place at8[4];  // rows 8g + row8 of the block
        int gq_c, i_c; // row c32
        const float *lse_b = a.lse + ((long long)b * a.Hq + (long long)k * a.G) * a.S;
        const float *delta_b = HAS_DELTA ? g.delta + ((long long)b * a.Hkv + k) * a.S * a.G : nullptr; // see delta_index
        auto fetch = [&](int rl0, BlockIn &x, uintx4 (&orow)[HAS_DELTA ? 1 : 4]) {
            const int rl = rl0 + X.c32 < nrows ? rl0 + X.c32 : nrows - 1; // (clamped: a valid row, whose <dout,out> is there)
            x.lse_row = lse_b[gq_c * a.S + i_c];
            x.drow = 0.f;
            if constexpr (HAS_DELTA) // left there by the dq kernel
                x.drow = delta_b[rl];
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                x.qr[g4] = *reinterpret_cast<const uintx4 *>(qb + at8[g4].q);
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                x.dor[g4] = *reinterpret_cast<const uintx4 *>(dob + at8[g4].o);
                if constexpr (!HAS_DELTA)
                    orow[g4] = *reinterpret_cast<const uintx4 *>(outb + at8[g4].o);
            }
        };
        // The last block (its rows past the candidate's clamped into it) and the one below it.
        auto place_block = [&](int rl0) {
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const int rl = rl0 + 8 * g4 + row8;
                place(rl < nrows ? rl : nrows - 1, at8[g4]);
            }
            const int rl = rl0 + X.c32 < nrows ? rl0 + X.c32 : nrows - 1;
            i_c = (int)fdiv((unsigned)rl, a.div_g);
            gq_c = rl - i_c * a.G;
        };
        auto step_down = [&] {
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                at8[g4].gq -= step_g;
                at8[g4].q -= step_q;
                at8[g4].o -= step_o;
                const bool neg = at8[g4].gq < 0;
                at8[g4].gq += neg ? a.G : 0;
                at8[g4].q += neg ? borrow_q : 0;
                at8[g4].o += neg ? borrow_o : 0;
            }
            gq_c -= step_g;
            i_c -= step_i;
            if (gq_c < 0) {
                gq_c += a.G;
                i_c -= 1;
            }
        };
        // The blocks that hold a row with i >= k0, from the candidate's last block down to the first
        // such one: the units of one (candidate, KV head) pair run side by side on one XCD (see the
        // kernel), and walking downwards they all ask for the same rows of q and dout at about the same
        // time, whatever their tile, so that those rows come from HBM once and from that XCD's L2 after.
        const int rl_first = (k0 * a.G) / kBlockRows * kBlockRows;
        const int rl_last = (nrows - 1) / kBlockRows * kBlockRows;
        // With <dout,out> at hand (no rows of out to fetch) there are registers to spare: the next
        // block is requested while the current one is worked on.
        constexpr bool kAhead = HAS_DELTA;
        BlockIn nx;
        uintx4 orow[HAS_DELTA ? 1 : 4];
        place_block(rl_last);
        int ri = i_c; // position of row c32 of the block being worked on
        bool first = true;
        if constexpr (kAhead) {
            fetch(rl_last, nx, orow);
            if (rl_last > rl_first)
                place_block(rl_last - kBlockRows);
        }
        for (int rl0 = rl_last; rl0 >= rl_first; rl0 -= kBlockRows) {
            if constexpr (!kAhead) {
                fetch(rl0, nx, orow);
                ri = i_c;
                if (first)
                    place_block(rl0 >= kBlockRows ? rl0 - kBlockRows : 0);
                else
                    step_down();
                first = false;
            }
            // row quantities, from where each lane fetches those of the rows its elements belong to
            if (X.h == 0) {
                aux_lse[X.c32] = nx.lse_row * kLog2e;
                aux_i[X.c32] = rl0 + X.c32 < nrows ? (float)ri : -1.f;
                if constexpr (HAS_DELTA)
                    aux_drow[X.c32] = nx.drow;
            }
            half_put(hp, img_q, nx.qr);
            half_put(hp, img_o, nx.dor);
            scratch_fence();
            if constexpr (!HAS_DELTA) {
                // this wavefront's 64 columns: all eight lanes of a row get its sum, one of them hands it on
                float p4[4];
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4)
                    p4[g4] = sum8(chunk_dot(nx.dor[g4], orow[g4]));
                const float mine = X.lane & 2 ? (X.lane & 1 ? p4[3] : p4[2]) : (X.lane & 1 ? p4[1] : p4[0]);
                if ((X.lane & 4) == 0)
                    xdrow[DH * 32 + 8 * (X.lane & 3) + row8] = mine;
            }
            if constexpr (kAhead) {
                // (past the end: the last block once more, so that nothing here depends on the loop's count)
                fetch(rl0 - kBlockRows >= rl_first ? rl0 - kBlockRows : rl0, nx, orow);
                ri = i_c;
                if (rl0 - 2 * kBlockRows >= rl_first)
                    step_down();
            }

            floatx16 s, dp;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                s[e] = 0.f;
                dp[e] = 0.f;
            }
            // this half of the two sums over the columns
#pragma unroll
            for (int i = 0; i < 4; ++i)
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(half_row_frag(hp, img_q, i)), as_bf16x8(kfh[i]), s, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(half_row_frag(hp, img_o, i)), as_bf16x8(vfh[i]), dp, 0, 0, 0);
            // The halves change hands.  Each wavefront completes S and dP for one of the block's two
            // 16-row steps only (wavefront DH: rows 16*DH .. 16*DH+15, accumulator elements 8*DH .. 8*DH+7):
            // it hands over its half of the other step's sums and later receives that step's finished
            // weights, so that the exponentials are taken once per element and not once per wavefront.
#pragma unroll
            for (int i2 = 0; i2 < 2; ++i2) {
                const int e0 = 4 * (2 * (1 - DH) + i2); // elements of the other wavefront's step
                *(lds_f32x4 *)(xch_mine + i2 * 1024) = floatx4{s[e0], s[e0 + 1], s[e0 + 2], s[e0 + 3]};
                *(lds_f32x4 *)(xch_mine + 2048 + i2 * 1024) = floatx4{dp[e0], dp[e0 + 1], dp[e0 + 2], dp[e0 + 3]};
            }
            __syncthreads();
            float sf[8], dpf[8];
#pragma unroll
            for (int i2 = 0; i2 < 2; ++i2) {
                const int e0 = 4 * (2 * DH + i2);
                const floatx4 so = *(lds_f32x4 *)(xch_other + i2 * 1024), dpo = *(lds_f32x4 *)(xch_other + 2048 + i2 * 1024);
#pragma unroll
                for (int t2 = 0; t2 < 4; ++t2) {
                    // the halves are added in a fixed order (columns 0..63 first), whichever wavefront does it
                    sf[4 * i2 + t2] = DH == 0 ? s[e0 + t2] + so[t2] : so[t2] + s[e0 + t2];
                    dpf[4 * i2 + t2] = DH == 0 ? dp[e0 + t2] + dpo[t2] : dpo[t2] + dp[e0 + t2];
                }
            }
            float p[8], ds[8];
#pragma unroll
            for (int i2 = 0; i2 < 2; ++i2) {
                const int kk = 2 * DH + i2;
                const floatx4 l4 = *(lds_f32x4 *)(aux_lse + 8 * kk + 4 * X.h);
                const floatx4 d4 = HAS_DELTA ? *(lds_f32x4 *)(aux_drow + 8 * kk + 4 * X.h)
                                             : *(lds_f32x4 *)(xdrow + 8 * kk + 4 * X.h) + *(lds_f32x4 *)(xdrow + 32 + 8 * kk + 4 * X.h);
                const floatx4 i4 = *(lds_f32x4 *)(aux_i + 8 * kk + 4 * X.h);
#pragma unroll
                for (int t2 = 0; t2 < 4; ++t2) {
                    const int e = 4 * i2 + t2;
                    // the row sees suffix key `key` iff key <= its position (which also means that the key exists)
                    const bool vis = (float)key <= i4[t2];
                    p[e] = vis ? fast_exp2(__builtin_fmaf(sf[e], X.c, -l4[t2])) : 0.f;
                    ds[e] = p[e] * (dpf[e] - d4[t2]);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // this step's packed weights and score gradients go to the other wavefront, the other step's come back
            uintx4 pfp_u[2], pfs_u[2];
            pfp_u[DH] = uintx4{pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]), pack_bf16(p[4], p[5]), pack_bf16(p[6], p[7])};
            pfs_u[DH] = uintx4{pack_bf16(ds[0], ds[1]), pack_bf16(ds[2], ds[3]), pack_bf16(ds[4], ds[5]), pack_bf16(ds[6], ds[7])};
            *(lds_u128 *)(xch_mine + 4096) = pfp_u[DH];
            *(lds_u128 *)(xch_mine + 4096 + 1024) = pfs_u[DH];
            // dO^T and Q^T for the second products: read here, they are there when the weights are
            bf16x8 at[2][2][2];
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i2 = 0; i2 < 2; ++i2) {
                    at[j][0][i2] = half_col_frag(hp, img_o, i2, j);
                    at[j][1][i2] = half_col_frag(hp, img_q, i2, j);
                }
            __syncthreads(); // also: the other wavefront has read this block's sums before the next block's are written
            pfp_u[1 - DH] = *(lds_u128 *)(xch_other + 4096);
            pfs_u[1 - DH] = *(lds_u128 *)(xch_other + 4096 + 1024);
            const bf16x8 pfp[2] = {as_bf16x8(pfp_u[0]), as_bf16x8(pfp_u[1])}, pfs[2] = {as_bf16x8(pfs_u[0]), as_bf16x8(pfs_u[1])};
            // the second products: this half of the columns of dV^T and dK^T
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i2 = 0; i2 < 2; ++i2) {
                    dv[i2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at[j][0][i2], pfp[j], dv[i2], 0, 0, 0);
                    dk[i2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at[j][1][i2], pfs[j], dk[i2], 0, 0, 0);
                }
            // (No barrier here: what this wavefront writes next for the other one - the next block's sums - is
            // read by it after the next barrier only, and it has read this block's before it reached the last one.)
        }
    }
    const bool kvalid = key < len;
    // where this lane's rows of the gradients go (worked out here, not before the loop: no registers held across it)
    unsigned short *dst_k[4], *dst_v[4];
    bool dst_ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int jr = k0 + 8 * u + (X.lane >> 3);
        dst_ok[u] = jr < a.S;
        const long long off = (long long)b * a.ks_sb + (long long)(dst_ok[u] ? jr : 0) * a.ks_ss + (long long)k * a.ks_sh +
                              8 * (X.lane & 7);
        dst_k[u] = reinterpret_cast<unsigned short *>(g.dk) + off;
        dst_v[u] = reinterpret_cast<unsigned short *>(g.dv) + off;
    }
    // the store routine addresses accumulators by column group: hand it this half in its place
    const floatx16 dk4[4] = {dk[0], dk[1], dk[0], dk[1]}, dv4[4] = {dv[0], dv[1], dv[0], dv[1]};
    store_rows<DH, DH>(X, dst_k, dst_ok, kvalid, a.scale, dk4);
    store_rows<DH, DH>(X, dst_v, dst_ok, kvalid, 1.0f, dv4);
}

template <bool HAS_DELTA, bool FIT>
__global__ __attribute__((amdgpu_flat_work_group_size(kDkvWaves * 64, kDkvWaves * 64), amdgpu_waves_per_eu(2, 4)))
void bwd_dkv_mfma_kernel(BwdArgs g, int nkt, int down)
{
    extern __shared__ __align__(256) unsigned char smem_generic[];
    lds_u8 *smem = (lds_u8 *)smem_generic;
    const int tid = threadIdx.x;
    // One unit - (candidate, KV head, 32-key tile) - per workgroup, one half of the output columns per
    // wavefront.  Workgroup ids go round the XCDs: the tiles of one (candidate, KV head) pair take
    // consecutive ids on ONE of them, so that they run there at the same time and share its L2.
    const int x = blockIdx.x & 7, y = blockIdx.x >> 3;
    const int grp = y / nkt, kt = y - grp * nkt;
    long long bk = (long long)grp * 8 + x;
    const long long pairs = (long long)g.f.B * g.f.Hkv;
    if (bk >= pairs) // the pairs are padded to a multiple of 8 (the same for the whole workgroup)
        return;
    bk = down ? pairs - 1 - bk : bk;
    // (wave-uniform branch; both sides meet the same workgroup barriers the same number of times)
    if (__builtin_amdgcn_readfirstlane(tid >> 6))
        bwd_dkv_unit<1, HAS_DELTA, FIT>(g, smem, tid, (int)bk, kt);
    else
        bwd_dkv_unit<0, HAS_DELTA, FIT>(g, smem, tid, (int)bk, kt);
}

} // namespace

bool bwd_mfma_supported(const Args &a, int dtype)
{
    return mfma_supported(a, dtype);
}

hipError_t launch_bwd_dkv_mfma(const BwdArgs &g, hipStream_t stream)
{
    const Args &a = g.f;
    const int nkt = (a.S + kTileKeys - 1) / kTileKeys;
    const long long nunits = ((long long)a.B * a.Hkv + 7) / 8 * 8 * nkt; // one workgroup each; pairs padded to a multiple of 8
    if (nunits > 0x7fffffffLL)
        return hipErrorInvalidValue;
    const bool fit = block_offsets_fit(a);
    auto kernel = g.delta ? (fit ? bwd_dkv_mfma_kernel<true, true> : bwd_dkv_mfma_kernel<true, false>)
                          : (fit ? bwd_dkv_mfma_kernel<false, true> : bwd_dkv_mfma_kernel<false, false>);
    // Where the tensors of query rows are twice the last-level cache (256 MB) and more, the pairs go from the last one down: what the
    // dq kernel has just read, the last candidates' q and dout, is still there.  us for the whole backward pass, upwards and
    // downwards: 1024 candidates x 16..24 positions x 4 heads, 8 KV heads, P 256 (805 MB of q, dout, out and dq): 300, 294; 1045
    // x 31 x 7, 4 KV heads, P 52 (930 MB): 326, 316; 244 x 77 x 4, 8 KV heads, P 203 (615 MB): 286, 280; 589 x 25 x 7,
    // 4 KV heads, P 753 (422 MB): 326, 325; 82 x 25 x 4, 8 KV heads, P 43 (67 MB): 28.9, 29.5.
    const int down = (double)a.B * a.S * a.Hq * a.D * 2 * 4 > 512e6;
    return launch_kernel(kernel, dim3((unsigned)nunits), dim3(kDkvWaves * 64), kDkvLdsBytes, stream, g, nkt, down);
}

hipError_t noalloc_scratch(void **ptr)
{
    static std::mutex mu;
    static void *by_device[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    if (dev < 0 || dev >= kMaxDevices)
        return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(mu);
    if (!by_device[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return e;
        if (!p)
            return hipErrorInvalidSymbol;
        by_device[dev] = p;
    }
    *ptr = by_device[dev];
    return hipSuccess;
}

hipError_t launch_bwd_dq_mfma(const BwdArgs &g, hipStream_t stream)
{
    static DeviceSlots cu_by_device;
    hipError_t e;
    const int num_cu = device_setup_once(cu_by_device, e, [] {
        hipError_t s = hipFuncSetAttribute(reinterpret_cast<const void *>(bwd_dq_mfma_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kBwdLdsBytes);
        for (auto kernel : {bwd_dq_packed_kernel<2>, bwd_dq_packed_kernel<1>})
            if (s == hipSuccess)
                s = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        2 * kDqMaxTiles * kTileBytes + kNW * kScrBytes);
        if (s == hipSuccess)
            s = hipFuncSetAttribute(reinterpret_cast<const void *>(bwd_dq_resident_kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                    2 * kDqMaxTiles * kTileBytes + kNW * kScrBytes);
        return s;
    });
    if (num_cu == 0)
        return e;
    const Args &a = g.f;
    const long long rows = (long long)a.C * a.S * a.G, rows_c = (long long)a.S * a.G;
    const long long nb = (rows_c + kBlockRows - 1) / kBlockRows; // blocks per candidate
    const bool fit = block_offsets_fit(a);
    // Short prefixes may stay resident in LDS (the split of the workgroups over the (instruction, KV
    // head) pairs is that of the resident forward kernel).  A candidate's last block may be partly empty, its only
    // one mostly: down to three rows in eight (12 rows per candidate, P 128: 158 us for the whole backward pass,
    // 162 us with the streaming kernel, whose blocks are full but span candidates; 8 rows: 146 and 132 us;
    // 20 rows: 217 and 242 us).
    const bool resident = a.P <= kDqMaxTiles * kTileKeys && rows_c * 8 >= nb * kBlockRows * 3 && fit && a.C * nb <= 0x7fffffffLL / 2;
    const ResidentSplit split = resident_split(a, a.C * nb, kNW, num_cu);
    // Rows packed by their lengths, where there are lengths: all of the resident kernel's calls and those of the streaming one up to 256 prefix
    // rows; calls of fewer than three blocks per wavefront that fill passes of four (below) stay with those.  us for the whole
    // backward pass, in those and so: 1024 x 16..24, 32/8 heads, P 256: 299, 281; 500 x 20, P 250: 152, 140; 500 x 14..28: 172, 151; 700 x 14..28, P 128:
    // 203, 188; 700 x 32..64: 480, 466; 700 x 10, 32/32: 223, 180; 32 x 10, 32/8: 19.0, 16.2; 32 x 28: 19.7, 20.9 (passes); nothing to pack: 700 x 32, 32/32: 430,
    // 431; 500 x 48, 28/4, P 250: 300, 307.
    const int max_tiles = (a.P + kTileKeys - 1) / kTileKeys;
    PackedArgs pa;
    const bool small = split.each < 3 && nb * 5 >= (nb + kUnitWaves - 1) / kUnitWaves * kUnitWaves * 4;
    if (const ResidentSplit packed = resident_split(a, a.C * nb * kNW, kNW, num_cu);
        a.len && !small && a.P <= kDqMaxTiles * kTileKeys && a.S <= 2 * kTileKeys && a.C * nb <= 0x7fffffffLL / kBlockRows &&
        (long long)a.P * a.kp_sp * 2 < 0x7fffffffLL && packed_args(a, (unsigned)packed.per_vh, kNW, pa)) {
        const bool two = packed_steps(a, 2, pa.dense) > 1;
        return launch_kernel(two ? bwd_dq_packed_kernel<2> : bwd_dq_packed_kernel<1>,
                             dim3((unsigned)(packed.per_vh * packed.vh_slots)), dim3(kNW * 64), (size_t)2 * max_tiles * kTileBytes + kNW * kScrBytes,
                             stream, DqPacked{g, pa, (int)packed.per_vh, (int)packed.vh_slots, max_tiles});
    }
    // Passes of four blocks of one candidate, where they come out full: at less than four blocks in five the
    // wavefronts without one cost more than sharing the tiles saves (five blocks in two passes, 40 positions x
    // 4 heads, P 128: 156 us against 130 us of the resident kernel and 141 us of the streaming one; four in one,
    // 27 x 4: 73 us, 91 us streamed; seven in two, 30 x 7: 153 us, 187 us streamed; 576 rows at P 128: 600 us for
    // the whole backward pass, 675 us without it).  They fetch the prefix once per pass, the resident kernel once per
    // launch: it is the better one where its wavefronts take three blocks or more and the passes, in rounds
    // of the chip against blocks per wavefront, make up more than 9/11 of the blocks' keys by their prefixes.  us for
    // the whole backward pass, passes and resident: 32 positions x 4 heads, 8 KV heads, P 256: 1024 candidates: 496,
    // 431; 512: 250, 232; 64: 31, 33; P 128, 512: 209, 215; P 64, 512: 192, 208; 30 x 7, 4 KV heads, 512
    // candidates, P 256: 205, 173; P 64: 145, 141; 144 x 4, 8 KV heads, 128 candidates, P 256: 355, 325; P 64: 272, 286.
    {
        UnitShape us;
        us.npc = (int)((nb + kUnitWaves - 1) / kUnitWaves);
        const long long npasses = ((long long)a.B * a.Hkv + 7) / 8 * 8 * us.npc;
        const long long rounds = (npasses + 2 * num_cu - 1) / (2 * num_cu);
        const bool stay = resident && split.each >= 3 && rounds * a.P * 11 > split.each * (a.P + (a.S + kTileKeys) / 2) * 9;
        if (!stay && fit && nb * 5 >= (long long)us.npc * kUnitWaves * 4 && npasses <= 0x7fffffffLL - 2 * num_cu) {
            us.div_npc = make_fastdiv((unsigned)us.npc);
            us.div_hkv = make_fastdiv((unsigned)a.Hkv);
            const unsigned grid = (unsigned)(npasses < 2 * num_cu ? npasses : 2 * num_cu);
            return launch_kernel(bwd_dq_unit_kernel, dim3(grid), dim3(kUnitWaves * 64), kUnitLdsBytes, stream, g, us, (int)npasses);
        }
    }
    if (resident) {
        const size_t lds = (size_t)2 * max_tiles * kTileBytes + kNW * kScrBytes;
        return launch_kernel(bwd_dq_resident_kernel, dim3((unsigned)(split.per_vh * split.vh_slots)), dim3(kNW * 64), lds, stream, g, (int)nb,
                             make_fastdiv((unsigned)nb), (int)split.per_vh, (int)split.vh_slots, max_tiles);
    }
    const long long npasses = ((rows + kBwdPassRows - 1) / kBwdPassRows) * a.Np * a.Hkv;
    // two workgroups fit a compute unit's LDS; registers allow one, so one per compute unit
    const unsigned grid = (unsigned)(npasses < num_cu ? npasses : num_cu);
    return launch_kernel(bwd_dq_mfma_kernel, dim3(grid), dim3(kNW * 64), kBwdLdsBytes, stream, g, (int)npasses);
}

} // namespace pskv
