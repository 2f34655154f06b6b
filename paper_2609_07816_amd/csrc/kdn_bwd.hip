// Backward pass of the chunked KDN forward (both variants) on gfx950.
//
// The forward's loss gradient is taken through its two stages (App. "Hardware-Efficient
// Chunkwise Algorithm": the gain scan, then the memory scan):
//
//  memory scan, given the gains kappa_t = G_t (.) k_t / c_t (G = p_hat and c the gain denominator
//  for the diagonal variant, G = beta and c = 1 for the isotropic one). Within a chunk of C tokens
//  with start state S_in and decays gamma_t = prod_{s <= t} alpha_s:
//      L = I + tril(M, -1),  M_ts = sum_i k_ti (gamma_t / gamma_s)_i kappa_si,
//      A_qk = tril(M^q) (q in place of k, diagonal included),  P_s = (gamma_C / gamma_s) kappa_s,
//      X = V - Kbar S_in,  Delta = L^-1 X,
//      O = scale (Qbar S_in + A_qk L^-1 X),  S_out = diag(gamma_C) S_in + KA^T X,  KA = L^-T P,
//  with Kbar = gamma k, Qbar = gamma q (eqs. chunk-memory-normalization to
//  chunk-memory-output-state). The forward leaves the division by c to L's diagonal; here Delta
//  itself is needed, and c times a row of that inverse has no value where c is infinite (r = inf,
//  a token without an observation: kappa = 0). Its adjoint, with dS_out from the chunk after:
//      Psi = dV = (A_qk L^-1)^T scale dO + KA dS_out,
//      dS_in = diag(gamma_C) dS_out + Qbar^T scale dO - Kbar^T Psi.
//  L^-1 is folded into KA and A_qk L^-1 once per chunk, so that both walks carry their state with
//  two products per chunk (Kbar then KA^T, KA then Kbar^T) and the rest is chunk-parallel.
//
//  gain scan. kappa_t = p_hat_t k_t / (r_t + sum_i p_hat_ti k_ti^2) (diagonal) or beta_t k_t
//  (isotropic), p_hat_t = alpha_t^2 p_{t-1} + omega_t (or a_t b_{t-1} + omega_t) and
//  p_t = p_hat_t / (1 + u_t p_hat_t) (eqs. kla-box-gain, diag-cov-update; iso-kla-box-gain,
//  iso-kla-box-cov-update). The adjoint of p_t obeys a linear recurrence backwards in time,
//  lambda_{t-1} = A_t lambda_t + B_t, whose coefficients are token-local; it is run per channel in
//  reverse, and every other gradient of the gain stage is token-local given it.
//
// Kernels, in launch order (summary and carry scan are the forward's):
//   bw_prep   per (chunk, head): variance replay from the carry, then the chunk's record
//   bw_fwalk  per (sequence, head, value tile): S_in of every chunk, X
//   bw_rwalk  per (sequence, head, value tile), chunks in reverse: dS_out, dV, dS0
//   bw_grad   per (chunk, head): dq, dk (memory part), dkappa, d(log-decay) -> dalpha part,
//             the coefficients of the variance adjoint
//   bw_scan   per (sequence, head, variance channel): the variance adjoint, dP0
//   bw_final  per (chunk, head): dk, dalpha, domega, dr of the gain stage
// Everything is float32 arithmetic; gradients are float32.
//
// Layouts between the kernels. A 16 x 16 float32 tile is 1 KB. In "lane order" it is 64 float4
// pieces, lane (g, i) = (lane / 16, lane % 16) holding rows 4 g .. 4 g + 3 of column i (an MFMA
// result tile, and the operand of a product that contracts over the rows) or columns
// 4 g .. 4 g + 3 of row i (the operand of one that contracts over the columns): one contiguous
// 1 KB read or write per wave. Matrices that both walks read, one along the rows and one along
// the columns, are kept as row-major tiles: either orientation touches the tile's 1 KB only.
#include "kdn_fwd.h"

namespace kdn {
namespace bwd {

using fwd::C;
using fwd::NB;
using fwd::SL;
constexpr int NTH = 256;  // four waves
constexpr int NLT = 10;   // lower 16 x 16 tiles of a C x C matrix, row by row
constexpr int LDL = 20;   // row-major 16 x 16 LDS tiles, rows padded to 80 bytes
// floor of the decay products inverted by the block-midpoint references: past it a factor
// saturates at 2^100
constexpr float DMIN = 0x1p-100f;

__device__ __forceinline__ constexpr int ltile(int b, int c) { return b * (b + 1) / 2 + c; }

// acc += A B for 16 x 16 operands in lane order (A: row i, columns 4 g ..; B: column i, rows
// 4 g ..): four 16 x 16 x 4 float32 MFMAs.
__device__ __forceinline__ floatx4 mm(floatx4 acc, floatx4 a, floatx4 b)
{
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], acc, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], acc, 0, 0, 0);
}

// N independent products step by step: a step on a result waits longer for the step before it than
// the unit takes per step, so consecutive ones go to different results.
template <int N>
__device__ __forceinline__ void mmn(floatx4 (&acc)[N], const floatx4 (&a)[N], const floatx4 (&b)[N])
{
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < N; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[i][e], acc[i], 0, 0, 0);
}

// a * s + b. The products that join a running value are summed from zero and added here: summed
// onto it, each of their steps would round at its size.
__device__ __forceinline__ floatx4 fma4(floatx4 a, float s, floatx4 b)
{
    return floatx4{fmaf(a[0], s, b[0]), fmaf(a[1], s, b[1]), fmaf(a[2], s, b[2]),
                   fmaf(a[3], s, b[3])};
}
__device__ __forceinline__ floatx4 fma4(floatx4 a, floatx4 s, floatx4 b)
{
    return floatx4{fmaf(a[0], s[0], b[0]), fmaf(a[1], s[1], b[1]), fmaf(a[2], s[2], b[2]),
                   fmaf(a[3], s[3], b[3])};
}

template <int N, int STRIDE = 1>
__device__ __forceinline__ floatx4 sum_parts(const floatx4* p)
{
    if constexpr (N == 4) return (p[0] + p[STRIDE]) + (p[2 * STRIDE] + p[3 * STRIDE]);
    else if constexpr (N == 2) return p[0] + p[STRIDE];
    else return p[0];
}

__device__ __forceinline__ floatx4 ldv(const float* p)
{
    return *reinterpret_cast<const floatx4*>(p);
}
__device__ __forceinline__ void stv(float* p, floatx4 v) { *reinterpret_cast<floatx4*>(p) = v; }

// A row-major 16 x 16 tile (16 floats per row) as an operand: by rows (lane (g, i): row i,
// columns 4 g ..) or by columns (rows 4 g .. of column i).
__device__ __forceinline__ floatx4 tile_rows(const float* t, int li, int lg)
{
    return ldv(t + 16 * li + 4 * lg);
}
__device__ __forceinline__ floatx4 tile_cols(const float* t, int li, int lg)
{
    const float* p = t + 64 * lg + li;
    return floatx4{p[0], p[16], p[32], p[48]};
}

__device__ __forceinline__ float inv_decay(float x)
{
    return __builtin_amdgcn_rcpf(fmaxf(x, DMIN));
}

// Per (chunk, head) record written by bw_prep (float32; tiles of 256 floats, sizes in floats).
template <int DK>
struct BwRec {
    static constexpr int NKT = DK / 16, TL = 256;
    static constexpr size_t NK = 0;                                 // -Kbar [4][NKT], row-major
    static constexpr size_t KA = NK + (size_t)4 * NKT * TL;         // KA [4][NKT], row-major
    static constexpr size_t QB = KA + (size_t)4 * NKT * TL;         // Qbar [4][NKT], columns
    static constexpr size_t LI = QB + (size_t)4 * NKT * TL;         // L^-1 [NLT], rows
    static constexpr size_t BA = LI + (size_t)NLT * TL;             // A_qk L^-1 [NLT], columns
    static constexpr size_t GC = BA + (size_t)NLT * TL;             // gamma_C [DK]
    static constexpr size_t DEN = GC + DK;                          // gain denominators [C]
    // diagonal: p_hat [4][NKT] by columns, then p before the chunk [DK];
    // isotropic: b_hat [C], then b before each token [C]
    static constexpr size_t PH = DEN + C;
    static constexpr size_t PP_D = PH + (size_t)4 * NKT * TL, PP_I = PH + C;
    static constexpr size_t size(bool diag)
    {
        return al256((diag ? PP_D + DK : PP_I + C) * 4) / 4;
    }
};

// Workspace of one backward call.
struct BwMap {
    size_t choff, summ, carry, rec, ckpt, xt, dso, dkp, dal, bcf, acf, aux, cmap, lpe, total;
    int maxch;
};

inline BwMap bw_map(int variant, bool packed, int N, int B, int T, int H, int dk, int dv,
                    size_t rec_floats)
{
    BwMap m;
    m.maxch = packed ? (int)((size_t)B * T / C + (size_t)N) : N * ((T + C - 1) / C);
    const size_t ch = (size_t)m.maxch * H;
    const size_t nchan = variant == 0 ? (size_t)dk : 1;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += al256(bytes);
        return o;
    };
    m.choff = take(packed ? (size_t)(N + 1) * 4 : 0);
    m.summ = take(ch * nchan * 16);
    m.carry = take(ch * nchan * 8);
    m.rec = take(ch * rec_floats * 4);
    m.ckpt = take(ch * dk * dv * 4);
    m.xt = take(ch * C * dv * 4);
    m.dso = take(ch * dk * dv * 4);
    m.dkp = take(ch * C * dk * 4);
    m.dal = take(ch * C * dk * 4);
    m.bcf = take(ch * C * nchan * 4);
    m.acf = take(variant == 0 ? 0 : ch * C * 4);
    m.aux = take(ch * C * 4 * (variant == 0 ? 1 : 2));
    m.cmap = take(ch * nchan * 8);
    m.lpe = take(ch * nchan * 4);
    m.total = off;
    return m;
}

struct Args {
    const void *q, *k, *v, *alpha, *omega, *r, *dO;
    const float *S0, *dS_T, *dP_T;
    float *dq, *dk, *dv, *dalpha, *domega, *dr, *dS0, *dP0;
    fwd::InArgs in;
    ChunkMap cm;
    int H, DV;
    uint32_t bytes_v, bytes_dv, bytes_dk;  // of v, of a float32 [.., H, DV], [.., H, DK]
    float mu, scale;
    const float2* carry;
    float* rec;        // [maxch][H] records of recn floats
    size_t recn;
    float* ckpt;       // S_in of every chunk: tiles [DK / 16][DV / 16] by rows (key), lane order
    float* xt;         // X: tiles [4][DV / 16] by columns (value), lane order
    float* dso;        // dS_out, laid out as ckpt
    float* dkp;        // dk without the variance adjoint's term: tiles [4][NKT] by columns
    float* dal;        // the log-decay part of dalpha: tiles [4][NKT] by columns
    float* bcf;        // diagonal: c_t with domega_t = lambda_t / (1 + u_t p_hat_t)^2 + c_t, tiles
                       // [4][NKT] by columns; isotropic: B_t [C]
    float* acf;        // isotropic: A_t [C]
    float* aux;        // diagonal: adjoint of the gain denominator [C]; isotropic: dbeta, ||k||^2
    float2* cmap;  // per (chunk, head, variance channel): the chunk's reverse map of the adjoint
    float* lpe;    // per (chunk, head, variance channel): the adjoint at the chunk's end
};

template <class TI>
__device__ __forceinline__ float ld(const void* p, size_t i)
{
    return to_f32(((const TI*)p)[i]);
}

// Stored value of a float32 or bf16 tensor at a 32-bit byte offset of its descriptor.
template <class TI>
__device__ __forceinline__ float bld(rsrc_t r, uint32_t off)
{
    return Raw1<TI>::f32(Raw1<TI>::load(r, off));
}

// Element i of a float32 gradient, where ok: without a branch, which would make the waits of the
// loads in flight conservative (the unit drops a store past the descriptor's end).
__device__ __forceinline__ void store_row(rsrc_t r, bool ok, uint32_t i, float x)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r,
                                          (int)(ok ? i * 4 : 0xFFFFFFFCu), 0, 0);
}

// ------------------------------------------------------------------------------------------
// bw_prep: one workgroup per (chunk, head), wave w = block w of 16 tokens, lane = channel pair in
// the variance phases (as the forward's prep, in float32). The products M and M^q run through two
// operand tiles in LDS, K and Q taking turns in the first: 79 KB at DK = 128, so that two
// workgroups fit a CU (three tiles would leave one). Bound by its 0.9 GB of traffic and by VALU
// issue: 226 us at B4 T4096 H16 d128 bf16 (4.1 TB/s) against 655 us when the record held kappa,
// p_hat, p, the log-decays (float64) and three decayed operands, formed by exponentials.
// ------------------------------------------------------------------------------------------
template <class TI, int DK_, int VARIANT_, bool APC_>
struct PrepCfg : fwd::VarCfg<TI, DK_, VARIANT_, APC_> {
    static constexpr int DK = DK_, NKT = DK / 16;
    static constexpr size_t SZ_OP = (size_t)C * DK * 4;
    // at the end X0 holds P_tail, X1 the tiles of L^-1 (lane order) and of A_qk (row-major)
    static constexpr size_t SZ_X1 = cmax(SZ_OP, (size_t)NLT * 1024 + (size_t)NLT * 16 * LDL * 4);
    static constexpr size_t OFF_X0 = 0, OFF_X1 = SZ_OP;
    // lower tiles of L, then L^-1's diagonal ones over L's; the blocks' Moebius products alias them
    static constexpr size_t OFF_LF = OFF_X1 + SZ_X1;
    static constexpr size_t OFF_SG = OFF_LF + cmax((size_t)NLT * 16 * LDL * 4, (size_t)NB * DK * 16);
    static constexpr size_t OFF_R = OFF_SG + (size_t)NB * DK * 4;
    static constexpr size_t OFF_MR = OFF_R + (size_t)C * 4;
    static constexpr size_t TOTAL = al16(OFF_MR + (size_t)C * 4);
};

// Operand tile [C][DK] in LDS, pieces of four channels of one token in MFMA operand order:
// fragment (block, s) is 64 pieces, token i's channels 16 s + 4 g .. + 3 at piece
// 16 g + (i ^ ((4 s + g) & 7)). The exclusive-or spreads a token's pieces over the banks when
// the lanes (one channel pair each) store them, and a fragment stays one contiguous KB.
template <int NKT>
__device__ __forceinline__ void op_put(float* X, int blk, int j, int ch, float x, float y)
{
    const int s = ch >> 4, g = (ch >> 2) & 3;
    const int p = (blk * NKT + s) * 64 + 16 * g + (j ^ ((4 * s + g) & 7));
    *reinterpret_cast<float2*>(X + 4 * p + (ch & 3)) = make_float2(x, y);
}
template <int NKT>
__device__ __forceinline__ floatx4 op_frag(const float* X, int blk, int s, int li, int lg)
{
    return ldv(X + 4 * ((blk * NKT + s) * 64 + 16 * lg + (li ^ ((4 * s + lg) & 7))));
}

// Block (ib, jb) of a product of two operand tiles; with mid, its column side scaled per channel
// by the decay of the blocks between (mid0, and mid1 where two lie between).
template <int NKT>
__device__ __forceinline__ floatx4 op_prod(const float* X0, const float* X1, int ib, int jb,
                                           const float* mid0, const float* mid1, int li, int lg)
{
    constexpr int NP = NKT >= 4 ? 4 : NKT;
    floatx4 acc[NP];
#pragma unroll
    for (int s = 0; s < NKT; ++s) {
        floatx4 p = op_frag<NKT>(X1, jb, s, li, lg);
        if (mid0) p *= ldv(mid0 + 16 * s + 4 * lg);
        if (mid1) p *= ldv(mid1 + 16 * s + 4 * lg);
        acc[s % NP] = mm(s < NP ? zero4() : acc[s % NP], op_frag<NKT>(X0, ib, s, li, lg), p);
    }
    return sum_parts<NP>(acc);
}

template <class TI, class CF>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(2))) void bw_prep(Args a)
{
    using R = BwRec<CF::DK>;
    constexpr int DK = CF::DK, NP = CF::NP, NKT = CF::NKT;
    constexpr bool DIAG = CF::DIAG;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float* X0 = (float*)(smem + CF::OFF_X0);
    float* X1 = (float*)(smem + CF::OFF_X1);
    float* Lf = (float*)(smem + CF::OFF_LF);
    float4* segA = (float4*)(smem + CF::OFF_LF);  // [NB][DK], dead before Lf is written
    float* segG = (float*)(smem + CF::OFF_SG);
    float* s_r = (float*)(smem + CF::OFF_R);
    float* s_mr = (float*)(smem + CF::OFF_MR);

    const int H = a.H;
    const int g = (int)(blockIdx.x / H), h = (int)(blockIdx.x % H);
    int n, c0, c1;
    bool last;
    if (!locate_chunk<C>(a.cm, g, n, c0, c1, last)) return;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pc = min(lane, NP - 1), ch = 2 * pc;
    const bool vact = lane < NP;
    float* rec = a.rec + ((size_t)g * H + h) * a.recn;

    const fwd::Src sr = fwd::make_src<TI, CF>(a.in, h, ch);
    if (tid < C) fwd::load_r<TI, false>(a.in, sr, c0, c1, tid, s_r, s_mr);
    const int Lw = c1 - (c0 + SL * w);  // tokens of this block in the sequence (may be <= 0)
    float2 Kf[SL], Qf[SL], Af[SL], Wf[SL];
    {
        fwd::SegIn<TI, CF, true> in;
        fwd::load_seg(in, sr, (uint32_t)(c0 + SL * w));
#pragma unroll
        for (int j = 0; j < SL; ++j) {
            const fwd::TokIn x = fwd::tok_in<true>(in, j, Lw);
            Kf[j] = x.K;
            Qf[j] = x.Q;
            Af[j] = x.A;
            Wf[j] = x.W;
        }
    }
    __syncthreads();

    // ---- the block's Moebius and decay products (eq. chunk-gain-summary) ---------------------
    float kn[DIAG ? 1 : SL], ka[DIAG ? 1 : SL];  // isotropic: ||k||^2 and mean alpha^2
    {
        float m0[4] = {1.f, 0.f, 0.f, 1.f}, m1[4] = {1.f, 0.f, 0.f, 1.f};
        float2 gs = make_float2(1.f, 1.f);
#pragma unroll
        for (int j = 0; j < SL; ++j) {
            const float mr = s_mr[SL * w + j];
            if constexpr (DIAG) {
                mob_left(m0, Af[j].x * Af[j].x, Wf[j].x, Kf[j].x * Kf[j].x * mr);
                mob_left(m1, Af[j].y * Af[j].y, Wf[j].y, Kf[j].y * Kf[j].y * mr);
            } else {
                kn[j] = wave_sum(vact ? fmaf(Kf[j].x, Kf[j].x, Kf[j].y * Kf[j].y) : 0.f);
                if constexpr (CF::APC)
                    ka[j] = wave_sum(vact ? fmaf(Af[j].x, Af[j].x, Af[j].y * Af[j].y) : 0.f) *
                            (1.f / (float)DK);
                else
                    ka[j] = Af[j].x * Af[j].x;
                mob_left(m0, ka[j], Wf[j].x, kn[j] * mr * (1.f / (float)DK));
            }
            gs.x *= Af[j].x;
            gs.y *= Af[j].y;
            if ((j & 3) == 3) {
                rescale4(m0);
                if constexpr (DIAG) rescale4(m1);
            }
        }
        if (vact) {
            if constexpr (DIAG) {
                segA[w * DK + ch] = make_float4(m0[0], m0[1], m0[2], m0[3]);
                segA[w * DK + ch + 1] = make_float4(m1[0], m1[1], m1[2], m1[3]);
            } else if (lane == 0) {
                segA[w * DK] = make_float4(m0[0], m0[1], m0[2], m0[3]);
            }
            *reinterpret_cast<float2*>(segG + w * DK + ch) = gs;
        }
    }
    __syncthreads();

    // ---- carry into the block; decay before it (Gs) and after it (Gt) within the chunk ------
    float n0, d0, n1 = 0.f, d1 = 1.f;
    float2 Gs = make_float2(1.f, 1.f), Gt = make_float2(1.f, 1.f);
    {
        const size_t cidx = ((size_t)g * H + h) * CF::NCHAN;
        if constexpr (DIAG) {
            float2 z0 = a.carry[cidx + ch], z1 = a.carry[cidx + ch + 1];
            if (w == 0 && vact)
                *reinterpret_cast<float2*>(rec + R::PP_D + ch) =
                    make_float2(z0.x / z0.y, z1.x / z1.y);
#pragma unroll
            for (int b = 0; b < NB - 1; ++b)
                if (b < w) {
                    z0 = mat_vec(segA[b * DK + ch], z0);
                    z1 = mat_vec(segA[b * DK + ch + 1], z1);
                }
            n0 = z0.x; d0 = z0.y; n1 = z1.x; d1 = z1.y;
        } else {
            float2 z = a.carry[cidx];
#pragma unroll
            for (int b = 0; b < NB - 1; ++b)
                if (b < w) z = mat_vec(segA[b * DK], z);
            n0 = z.x; d0 = z.y;
        }
        float2 gc = make_float2(1.f, 1.f);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float2 gg = *reinterpret_cast<const float2*>(segG + b * DK + ch);
            if (b < w) { Gs.x *= gg.x; Gs.y *= gg.y; }
            if (b > w) { Gt.x *= gg.x; Gt.y *= gg.y; }
            gc.x *= gg.x;
            gc.y *= gg.y;
        }
        if (w == 0 && vact) *reinterpret_cast<float2*>(rec + R::GC + ch) = gc;
    }

    // ---- replay (eqs. chunk-gain-local-prefix, chunk-gain-emission): kappa_t per channel of the
    // pair; the gain denominators --------------------------------------------------------------
    // tiles by columns: a channel's four tokens 4 e .. + 3 of block w, its neighbour's beside them
    auto col_piece = [&](float* base, int e) {
        return base + ((size_t)(w * NKT + (ch >> 4)) * 64 + 16 * e + (ch & 15)) * 4;
    };
    float2 pk[SL];
    {
        float hx[4], hy[4];
#pragma unroll
        for (int j = 0; j < SL; ++j) {
            const int t = SL * w + j;
            if constexpr (DIAG) {
                const float mr = s_mr[t];
                const float nn0 = fmaf(Af[j].x * Af[j].x, n0, Wf[j].x * d0);  // p_hat d
                const float nn1 = fmaf(Af[j].y * Af[j].y, n1, Wf[j].y * d1);
                const float ph0 = nn0 * __builtin_amdgcn_rcpf(d0);
                const float ph1 = nn1 * __builtin_amdgcn_rcpf(d1);
                hx[j & 3] = ph0;
                hy[j & 3] = ph1;
                if ((j & 3) == 3 && vact) {
                    float* p = col_piece(rec + R::PH, j >> 2);
                    stv(p, floatx4{hx[0], hx[1], hx[2], hx[3]});
                    stv(p + 4, floatx4{hy[0], hy[1], hy[2], hy[3]});
                }
                pk[j] = make_float2(ph0 * Kf[j].x, ph1 * Kf[j].y);
                const float z = wave_sum(vact ? fmaf(pk[j].x, Kf[j].x, pk[j].y * Kf[j].y) : 0.f);
                // (r is 1 past the end, where z holds 0 times variances that may not be finite)
                const float dn = s_r[t] + (j < Lw ? z : 0.f), idn = __builtin_amdgcn_rcpf(dn);
                if (lane == 0) rec[R::DEN + t] = dn;
                pk[j].x *= idn;
                pk[j].y *= idn;
                d0 = fmaf(Kf[j].x * Kf[j].x * mr, nn0, d0);
                d1 = fmaf(Kf[j].y * Kf[j].y * mr, nn1, d1);
                n0 = nn0;
                n1 = nn1;
                if ((j & 3) == 3) {
                    rescale2(n0, d0);
                    rescale2(n1, d1);
                }
            } else {
                const float nn = fmaf(ka[j], n0, Wf[j].x * d0);  // b_hat d
                const float bh = j < Lw ? nn / d0 : 0.f;
                const float dn = fmaf(bh, kn[j], s_r[t]), beta = bh / dn;
                if (lane == 0) {
                    rec[R::PP_I + t] = n0 / d0;
                    rec[R::PH + t] = bh;
                    rec[R::DEN + t] = dn;
                }
                pk[j] = make_float2(beta * Kf[j].x, beta * Kf[j].y);
                d0 = fmaf(kn[j] * s_mr[t] * (1.f / (float)DK), nn, d0);
                n0 = nn;
                if ((j & 3) == 3) rescale2(n0, d0);
            }
        }
    }

    // ---- -Kbar (row-major tiles) and Qbar (by columns) ---------------------------------------
    if (vact) {
        float2 P = Gs;
        float qx[4], qy[4];
        float* nk = rec + R::NK + (size_t)(w * NKT + (ch >> 4)) * 256 + (ch & 15);
#pragma unroll
        for (int j = 0; j < SL; ++j) {
            P.x *= Af[j].x;
            P.y *= Af[j].y;
            *reinterpret_cast<float2*>(nk + 16 * j) = make_float2(-P.x * Kf[j].x, -P.y * Kf[j].y);
            qx[j & 3] = P.x * Qf[j].x;
            qy[j & 3] = P.y * Qf[j].y;
            if ((j & 3) == 3) {
                float* p = col_piece(rec + R::QB, j >> 2);
                stv(p, floatx4{qx[0], qx[1], qx[2], qx[3]});
                stv(p + 4, floatx4{qy[0], qy[1], qy[2], qy[3]});
            }
        }
    }

    // ---- diagonal blocks: operands referenced to the block midpoint (own rows only, so no
    // barrier between their stores and products). F_t = prod_{8 <= j <= t} alpha_j (t >= 8),
    // 1 / prod_{t < j <= 7} alpha_j (t < 8); K_t F_t and kappa_s / F_s give the ratio ---------
    auto put_mid = [&](float* X, const float2* x, bool inv) __attribute__((always_inline)) {
        float2 b = make_float2(1.f, 1.f);
#pragma unroll
        for (int j = SL / 2 - 1; j >= 0; --j) {
            const float fx = inv ? b.x : inv_decay(b.x), fy = inv ? b.y : inv_decay(b.y);
            op_put<NKT>(X, w, j, ch, x[j].x * fx, x[j].y * fy);
            b.x *= Af[j].x;
            b.y *= Af[j].y;
        }
        float2 f = make_float2(1.f, 1.f);
#pragma unroll
        for (int j = SL / 2; j < SL; ++j) {
            f.x *= Af[j].x;
            f.y *= Af[j].y;
            const float fx = inv ? inv_decay(f.x) : f.x, fy = inv ? inv_decay(f.y) : f.y;
            op_put<NKT>(X, w, j, ch, x[j].x * fx, x[j].y * fy);
        }
    };
    auto put_start = [&](float* X, const float2* x) __attribute__((always_inline)) {
        float2 P = make_float2(1.f, 1.f);
#pragma unroll
        for (int j = 0; j < SL; ++j) {
            P.x *= Af[j].x;
            P.y *= Af[j].y;
            op_put<NKT>(X, w, j, ch, x[j].x * P.x, x[j].y * P.y);
        }
    };
    if (vact) {
        put_mid(X0, Kf, false);
        put_mid(X1, pk, true);
    }
    __syncthreads();  // the blocks' Moebius products are dead: L's tiles over them
    auto lblk = [&](int b, int c) { return Lf + ltile(b, c) * 16 * LDL; };
    {
        const floatx4 t = op_prod<NKT>(X0, X1, w, w, nullptr, nullptr, li, lg);
        float* lb = lblk(w, w);
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int row = 4 * lg + rr;
            // (rows past the end, zeros times kappa, are zeros also where a kappa is not finite)
            lb[row * LDL + li] = row > li && row < Lw ? t[rr] : (row == li ? 1.f : 0.f);
        }
    }
    wave_lds_fence();
    if (vact) put_mid(X0, Qf, false);
    wave_lds_fence();
    floatx4 aqd = op_prod<NKT>(X0, X1, w, w, nullptr, nullptr, li, lg);
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) aqd[rr] = 4 * lg + rr >= li ? aqd[rr] : 0.f;

    // ---- blocks off the diagonal: rows referenced to their block's start, columns to their
    // block's end, the decay of the blocks between applied to the column side. Pairs per wave:
    // 0: (1,0) (3,0); 1: (2,1) (3,1); 2: (3,2) (2,0); 3: the diagonal blocks of L^-1 ----------
    wave_lds_fence();
    if (vact) {
        put_start(X0, Kf);
        float2 Q = make_float2(1.f, 1.f);
#pragma unroll
        for (int j = SL - 1; j >= 0; --j) {
            op_put<NKT>(X1, w, j, ch, pk[j].x * Q.x, pk[j].y * Q.y);
            Q.x *= Af[j].x;
            Q.y *= Af[j].y;
        }
    }
    __syncthreads();
    const int ib0 = w + 1, jb0 = w;                       // the wave's two pairs (w < 3)
    const int ib1 = w == 2 ? 2 : 3, jb1 = w == 1 ? 1 : 0;
    const float* mid0 = segG + (jb1 + 1) * DK;            // pair 1 is two or three apart
    const float* mid1 = w == 0 ? segG + 2 * DK : nullptr;
    if (w < 3) {
        auto put = [&](int b, int c, floatx4 t) {
            float* lb = lblk(b, c);
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) lb[(4 * lg + rr) * LDL + li] = t[rr];
        };
        put(ib0, jb0, op_prod<NKT>(X0, X1, ib0, jb0, nullptr, nullptr, li, lg));
        put(ib1, jb1, op_prod<NKT>(X0, X1, ib1, jb1, mid0, mid1, li, lg));
    } else {
        // Row i of A_bb = L_bb^-1 solves a^T L_bb = e_i^T: a_i = 1, and going down the rows
        // m = i, i-1, ..., 0 every finished a_m adds a_m L_m,k to the sums of the k < m
        // (right-looking backward substitution). Lane (b, i) takes row i of block b; the wave has
        // read every tile before it stores over them.
        float* Lb = lblk(lg, lg);
        float sacc[16], y[16];
#pragma unroll
        for (int kq = 0; kq < 16; ++kq) sacc[kq] = 0.f;
#pragma unroll
        for (int mq = 15; mq >= 0; --mq) {
            float cur[16];
#pragma unroll
            for (int v4 = 0; v4 < (mq + 3) / 4; ++v4) {
                const floatx4 q4 = ldv(Lb + mq * LDL + 4 * v4);
#pragma unroll
                for (int e = 0; e < 4; ++e) cur[4 * v4 + e] = q4[e];
            }
            y[mq] = mq > li ? 0.f : (mq == li ? 1.f : 0.f) - sacc[mq];
#pragma unroll
            for (int kq = 0; kq < mq; ++kq) sacc[kq] = fmaf(y[mq], cur[kq], sacc[kq]);
        }
        wave_lds_fence();
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4)
            stv(Lb + li * LDL + 4 * v4,
                floatx4{y[4 * v4], y[4 * v4 + 1], y[4 * v4 + 2], y[4 * v4 + 3]});
    }
    __syncthreads();
    if (vact) put_start(X0, Qf);
    __syncthreads();
    floatx4 aqo[2];
    if (w < 3) {
        aqo[0] = op_prod<NKT>(X0, X1, ib0, jb0, nullptr, nullptr, li, lg);
        aqo[1] = op_prod<NKT>(X0, X1, ib1, jb1, mid0, mid1, li, lg);
    }
    __syncthreads();

    // ---- L^-1 by columns of blocks: wave c takes block column c,
    // Li_bc = -A_bb sum_{c <= j < b} L_bj Li_jc, Li_cc = A_cc; A_qk and P_tail staged ---------
    float* s_li = X1;              // L^-1 [NLT] lane order (by columns)
    float* s_aq = X1 + NLT * 256;  // A_qk [NLT] row-major, LDL
    floatx4 lt[NB];
    {
        auto put = [&](int b, int c, floatx4 t) {
            float* p = s_aq + ltile(b, c) * 16 * LDL;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) p[(4 * lg + rr) * LDL + li] = t[rr];
        };
        put(w, w, aqd);
        if (w < 3) {
            put(ib0, jb0, aqo[0]);
            put(ib1, jb1, aqo[1]);
        }
        const int c = w;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            lt[b] = zero4();
            if (b == c) {
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) lt[b][rr] = lblk(c, c)[(4 * lg + rr) * LDL + li];
            } else if (b > c) {
                floatx4 acc = zero4();
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    if (j >= c && j < b) acc = mm(acc, ldv(lblk(b, j) + li * LDL + 4 * lg), lt[j]);
                lt[b] = -mm(zero4(), ldv(lblk(b, b) + li * LDL + 4 * lg), acc);
            }
            if (b >= c) stv(s_li + ltile(b, c) * 256 + 4 * lane, lt[b]);
        }
        if (vact) {  // P_tail = (gamma_C / gamma_s) kappa_s, by columns
            float px[4], py[4];
            float2 Q = Gt;
#pragma unroll
            for (int j = SL - 1; j >= 0; --j) {
                px[j & 3] = pk[j].x * Q.x;
                py[j & 3] = pk[j].y * Q.y;
                if ((j & 3) == 0) {
                    float* p = col_piece(X0, j >> 2);
                    stv(p, floatx4{px[0], px[1], px[2], px[3]});
                    stv(p + 4, floatx4{py[0], py[1], py[2], py[3]});
                }
                Q.x *= Af[j].x;
                Q.y *= Af[j].y;
            }
        }
    }
    __syncthreads();
    // L^-1 by rows: through L's tiles (dead), the wave's own columns
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if (b >= w) {
            float* p = lblk(b, w);
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) p[(4 * lg + rr) * LDL + li] = lt[b][rr];
        }
    wave_lds_fence();
#pragma unroll
    for (int b = 0; b < NB; ++b)
        if (b >= w)
            stv(rec + R::LI + ltile(b, w) * 256 + 4 * lane, ldv(lblk(b, w) + li * LDL + 4 * lg));
    // A_qk L^-1, row block w (by columns: the result tiles as they are)
#pragma unroll
    for (int sb = 0; sb < NB; ++sb)
        if (sb <= w) {
            floatx4 acc = zero4();
#pragma unroll
            for (int ub = 0; ub < NB; ++ub)
                if (ub >= sb && ub <= w)
                    acc = mm(acc, ldv(s_aq + ltile(w, ub) * 16 * LDL + li * LDL + 4 * lg),
                             ldv(s_li + ltile(ub, sb) * 256 + 4 * lane));
            stv(rec + R::BA + ltile(w, sb) * 256 + 4 * lane, acc);
        }
    // KA^T = P_tail^T L^-1 by channel tiles: the result (channel 4 g .., token i) is a row-major
    // tile of KA
    for (int ct = w; ct < NKT; ct += 4) {
        floatx4 pt[NB];
#pragma unroll
        for (int sb = 0; sb < NB; ++sb) pt[sb] = ldv(X0 + ((sb * NKT + ct) * 64 + lane) * 4);
#pragma unroll
        for (int tb = 0; tb < NB; ++tb) {
            floatx4 acc = zero4();
#pragma unroll
            for (int sb = tb; sb < NB; ++sb)
                acc = mm(acc, pt[sb], ldv(s_li + ltile(sb, tb) * 256 + 4 * lane));
            stv(rec + R::KA + (size_t)(tb * NKT + ct) * 256 + 16 * li + 4 * lg, acc);
        }
    }
}

// ------------------------------------------------------------------------------------------
// walks over the chunks of one (sequence, head, tile of 16 NJT value columns). Four waves: wave w
// owns row block w of the chunk (X, Psi) and key tiles KPW w .. of the state, which stays in its
// registers transposed (value rows, key columns), so that every state tile is stored as it is for
// bw_grad; the state, X or Psi and scale dO go through LDS as [value][key or token]. The record
// operands are read straight into registers, one chunk ahead. At DK = 128, NJT = 2 a chunk is
// 128 (forward) or up to 224 (reverse) MFMAs of 32 cycles per wave on its SIMD's matrix core.
// Every load is unconditional: with one inside a branch the compiler has to assume it was not
// issued and waits for the newest loads instead of the oldest. Each operand is fetched again right
// after the step that used it, between the MFMAs: issued in one burst before the barrier, the four
// waves' loads queue for the CU's one memory pipeline while no MFMA runs. At B4 T4096 H16 d128
// (one workgroup per CU, 64 chunks in series): 206 and 304 us, against 272 and 393 us with bursts
// and a product's dependent steps in sequence, and 589 and 721 us with the operands staged through
// LDS and L^-1 applied inside the walk (a third product and barrier per chunk).
// ------------------------------------------------------------------------------------------
template <int DK, int NJT>
struct WalkCfg {
    static constexpr int NKT = DK / 16, KPW = NKT >= 4 ? NKT / 4 : 1;
    static constexpr int BV = 16 * NJT, LDK = DK + 4, LDC = C + 4;
    static constexpr bool ALL = NKT >= 4;  // every wave owns key tiles
    // partial sums of a product over the keys: each is summed on its own, which shortens the
    // chains of roundings
    static constexpr int NP = NKT >= 4 ? 4 : NKT;
};

// Block -> (sequence-head slot, value tile): the NV tiles of one head get block indices
// congruent modulo 8, so round-robin dispatch puts them on one XCD, where they share the L2 copy
// of the head's chunk records. The grid is padded to a multiple of 8 slots.
__device__ __forceinline__ bool walk_slot(const Args& a, int NV, int& slot, int& vt)
{
    const int xcd = (int)(blockIdx.x % 8), rest = (int)(blockIdx.x / 8);
    vt = rest % NV;
    slot = (rest / NV) * 8 + xcd;
    return slot < a.cm.N * a.H;
}

template <class TI, int DK, int NJT>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(1))) void bw_fwalk(Args a)
{
    using R = BwRec<DK>;
    using CF = WalkCfg<DK, NJT>;
    constexpr int NKT = CF::NKT, KPW = CF::KPW, LDK = CF::LDK, LDC = CF::LDC, BV = CF::BV;
    __shared__ __attribute__((aligned(16))) float s_S[BV * LDK], s_X[BV * LDC];
    const int H = a.H, DV = a.DV, NJ = DV / 16;
    int slot, vt;
    if (!walk_slot(a, DV / BV, slot, vt)) return;
    const int n = slot / H, h = slot % H, j0 = vt * BV;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // first key tile of the wave; waves without one compute a copy of the last and store nothing,
    // so that no wave skips a load (a skipped one would make the others' waits conservative)
    const int kt0 = min(KPW * w, NKT - 1);
    const bool own = CF::ALL || w < NKT;
    int t0, t1, g0, nch;
    seq_span(a.cm, n, t0, t1);
    seq_chunks<C>(a.cm, n, t0, t1, g0, nch);
    if (nch == 0) return;
    const rsrc_t rv = make_rsrc(a.v, a.bytes_v);
    constexpr uint32_t es = sizeof(TI);
    const uint32_t rowv = (uint32_t)H * DV * es;
    const uint32_t colv = ((uint32_t)h * DV + j0 + li) * es;

    floatx4 S[KPW][NJT];
    auto put_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < KPW; ++u)
#pragma unroll
            for (int jt = 0; jt < NJT; ++jt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    s_S[(16 * jt + 4 * lg + r) * LDK + 16 * (kt0 + u) + li] = S[u][jt][r];
    };
#pragma unroll
    for (int u = 0; u < KPW; ++u)
#pragma unroll
        for (int jt = 0; jt < NJT; ++jt)
            S[u][jt] = a.S0 ? ldv(a.S0 + ((size_t)slot * DK + 16 * (kt0 + u) + li) * DV + j0 +
                                  16 * jt + 4 * lg)
                            : zero4();
    if (own) put_state();
    floatx4 kf[NKT], ka[KPW][NB];
    float gc[KPW];
    typename Raw1<TI>::type vr[NJT][4];
    auto recp = [&](int m) { return a.rec + ((size_t)(g0 + min(m, nch - 1)) * H + h) * a.recn; };
    auto load_k = [&](int m, int s) __attribute__((always_inline)) {
        kf[s] = tile_rows(recp(m) + R::NK + (size_t)(w * NKT + s) * 256, li, lg);
    };
    auto load_v = [&](int m) __attribute__((always_inline)) {
        const uint32_t c0 = (uint32_t)(t0 + min(m, nch - 1) * C + 16 * w + 4 * lg);
#pragma unroll
        for (int jt = 0; jt < NJT; ++jt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                vr[jt][r] = Raw1<TI>::load(rv, (c0 + r) * rowv + colv + 16 * jt * es);
    };
    auto load_a = [&](int m, int tb) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < KPW; ++u)
            ka[u][tb] = tile_cols(recp(m) + R::KA + (size_t)(tb * NKT + kt0 + u) * 256, li, lg);
    };
    auto load_g = [&](int m) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < KPW; ++u) gc[u] = recp(m)[R::GC + 16 * (kt0 + u) + li];
    };
    // the state tiles' product: m [value][token] (LDS) with the wave's key tiles of a record matrix;
    // reload(tb) fetches the next chunk's tiles of a step once it is done
    auto state_prod = [&](floatx4 (&up)[KPW * NJT], const float* m, const floatx4 (&t)[KPW][NB],
                          auto reload) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < KPW * NJT; ++i) up[i] = zero4();
#pragma unroll
        for (int tb = 0; tb < NB; ++tb) {
            floatx4 av[KPW * NJT], bv[KPW * NJT];
#pragma unroll
            for (int i = 0; i < KPW * NJT; ++i) {
                av[i] = ldv(m + (16 * (i % NJT) + li) * LDC + 16 * tb + 4 * lg);
                bv[i] = t[i / NJT][tb];
            }
            mmn(up, av, bv);
            reload(tb);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll
    for (int s = 0; s < NKT; ++s) load_k(0, s);
    load_v(0);
#pragma unroll
    for (int tb = 0; tb < NB; ++tb) load_a(0, tb);
    load_g(0);
    __syncthreads();
    for (int m = 0; m < nch; ++m) {
        const int L = min(C, t1 - (t0 + m * C));
        const size_t gh = (size_t)(g0 + m) * H + h;
        if (own) {  // checkpoint: S_in of this chunk
#pragma unroll
            for (int u = 0; u < KPW; ++u)
#pragma unroll
                for (int jt = 0; jt < NJT; ++jt)
                    stv(a.ckpt + (((gh * NKT + kt0 + u) * NJ + vt * NJT + jt) * 64 + lane) * 4,
                        S[u][jt]);
        }
        // X = V - Kbar S_in, row block w
        // partial sums by key tile modulo NP, [NP][NJT]
        floatx4 x[NJT], xp[CF::NP * NJT];
#pragma unroll
        for (int i = 0; i < CF::NP * NJT; ++i) xp[i] = zero4();
#pragma unroll
        for (int s = 0; s < NKT; s += CF::NP) {
            floatx4 av[CF::NP * NJT], bv[CF::NP * NJT];
#pragma unroll
            for (int i = 0; i < CF::NP * NJT; ++i) {
                const int st = s + i / NJT, jt = i % NJT;
                av[i] = kf[st];
                bv[i] = ldv(s_S + (16 * jt + li) * LDK + 16 * st + 4 * lg);
            }
            mmn(xp, av, bv);
#pragma unroll
            for (int i = 0; i < CF::NP; ++i) load_k(m + 1, s + i);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int jt = 0; jt < NJT; ++jt) {
            x[jt] = sum_parts<CF::NP, NJT>(xp + jt);
#pragma unroll
            for (int r = 0; r < 4; ++r)  // rows past the end of the sequence read as zeros
                x[jt][r] += 16 * w + 4 * lg + r < L ? Raw1<TI>::f32(vr[jt][r]) : 0.f;
            stv(s_X + (16 * jt + li) * LDC + 16 * w + 4 * lg, x[jt]);
            stv(a.xt + (((gh * 4 + w) * NJ + vt * NJT + jt) * 64 + lane) * 4, x[jt]);
        }
        load_v(m + 1);
        __syncthreads();
        // S^T <- S^T diag(gamma_C) + X^T KA
        {
            floatx4 up[KPW * NJT];
            state_prod(up, s_X, ka, [&](int tb) { load_a(m + 1, tb); });
#pragma unroll
            for (int u = 0; u < KPW; ++u)
#pragma unroll
                for (int jt = 0; jt < NJT; ++jt) S[u][jt] = fma4(S[u][jt], gc[u], up[u * NJT + jt]);
            if (own) put_state();
        }
        load_g(m + 1);
        __syncthreads();
    }
}

// (two waves per SIMD: uncapped it takes 258 registers at DK = 128, NJT = 2, and then one workgroup
// per CU, 18.7 against 16.2 us for one chunk of 128 sequence-heads; capped, one pair goes to scratch)
template <class TI, int DK, int NJT>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(2))) void bw_rwalk(Args a)
{
    using R = BwRec<DK>;
    using CF = WalkCfg<DK, NJT>;
    constexpr int NKT = CF::NKT, KPW = CF::KPW, LDK = CF::LDK, LDC = CF::LDC, BV = CF::BV;
    constexpr int PER = BV / 4;  // dO values per thread: token tid / 4, columns PER (tid % 4) ..
    __shared__ __attribute__((aligned(16))) float s_S[BV * LDK], s_P[BV * LDC], s_O[BV * LDC];
    const int H = a.H, DV = a.DV, NJ = DV / 16;
    int slot, vt;
    if (!walk_slot(a, DV / BV, slot, vt)) return;
    const int n = slot / H, h = slot % H, j0 = vt * BV;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kt0 = min(KPW * w, NKT - 1);
    const bool own = CF::ALL || w < NKT;
    int t0, t1, g0, nch;
    seq_span(a.cm, n, t0, t1);
    seq_chunks<C>(a.cm, n, t0, t1, g0, nch);

    floatx4 S[KPW][NJT];  // dS^T
    auto put_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < KPW; ++u)
#pragma unroll
            for (int jt = 0; jt < NJT; ++jt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    s_S[(16 * jt + 4 * lg + r) * LDK + 16 * (kt0 + u) + li] = S[u][jt][r];
    };
    auto state_at = [&](int u, int jt) {
        return ((size_t)slot * DK + 16 * (kt0 + u) + li) * DV + j0 + 16 * jt + 4 * lg;
    };
#pragma unroll
    for (int u = 0; u < KPW; ++u)
#pragma unroll
        for (int jt = 0; jt < NJT; ++jt)
            S[u][jt] = a.dS_T ? ldv(a.dS_T + state_at(u, jt)) : zero4();
    if (own) put_state();
    floatx4 ka[NKT], ba[NB], qb[KPW][NB], nk[KPW][NB];
    float gc[KPW];
    // dO as stored, and a mask of its rows: both are read when it is put to LDS, without a branch
    typedef unsigned OW __attribute__((ext_vector_type(PER * sizeof(TI) / 4)));
    OW ow = {};
    unsigned omask = 0;
    const rsrc_t rdv = make_rsrc(a.dv, a.bytes_dv);
    auto recp = [&](int m) { return a.rec + ((size_t)(g0 + max(m, 0)) * H + h) * a.recn; };
    auto load_a = [&](int m, int s) __attribute__((always_inline)) {
        ka[s] = tile_rows(recp(m) + R::KA + (size_t)(w * NKT + s) * 256, li, lg);
    };
    auto load_b = [&](int m, int tb) __attribute__((always_inline)) {
        ba[tb] = ldv(recp(m) + R::BA + ltile(max(tb, w), w) * 256 + 4 * lane);
    };
    auto load_o = [&](int m) __attribute__((always_inline)) {
        const int c0 = t0 + max(m, 0) * C, t = tid >> 2;
        const bool ok = a.dO && t < t1 - c0;
        // every thread loads: a row inside the sequence, v's where there is no dO
        const TI* p = (const TI*)(a.dO ? a.dO : a.v) +
                      ((size_t)(c0 + min(t, t1 - c0 - 1)) * H + h) * DV + j0 + PER * (tid & 3);
        __builtin_memcpy(&ow, __builtin_assume_aligned(p, sizeof(ow) < 16 ? sizeof(ow) : 16),
                         sizeof(ow));
        omask = ok ? ~0u : 0u;
    };
    auto put_o = [&]() __attribute__((always_inline)) {  // scale dO
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            float x;
            if constexpr (sizeof(TI) == 4) {
                x = __uint_as_float(ow[e] & omask);
            } else {
                const float2 y = unpack2(ow[e / 2] & omask);
                x = e & 1 ? y.y : y.x;
            }
            s_O[(PER * (tid & 3) + e) * LDC + (tid >> 2)] = a.scale * x;
        }
    };
    auto load_q = [&](int m, int tb) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < KPW; ++u)
            qb[u][tb] = ldv(recp(m) + R::QB + ((size_t)(tb * NKT + kt0 + u) * 64 + lane) * 4);
    };
    auto load_k = [&](int m, int tb) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < KPW; ++u)
            nk[u][tb] = tile_cols(recp(m) + R::NK + (size_t)(tb * NKT + kt0 + u) * 256, li, lg);
    };
    auto load_g = [&](int m) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < KPW; ++u) gc[u] = recp(m)[R::GC + 16 * (kt0 + u) + li];
    };
    // the state tiles' product: m [value][token] (LDS) with the wave's key tiles of a record matrix;
    // reload(tb) fetches the next chunk's tiles of a step once it is done
    auto state_prod = [&](floatx4 (&up)[KPW * NJT], const float* m, const floatx4 (&t)[KPW][NB],
                          auto reload) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < KPW * NJT; ++i) up[i] = zero4();
#pragma unroll
        for (int tb = 0; tb < NB; ++tb) {
            floatx4 av[KPW * NJT], bv[KPW * NJT];
#pragma unroll
            for (int i = 0; i < KPW * NJT; ++i) {
                av[i] = ldv(m + (16 * (i % NJT) + li) * LDC + 16 * tb + 4 * lg);
                bv[i] = t[i / NJT][tb];
            }
            mmn(up, av, bv);
            reload(tb);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (nch > 0) {
        load_o(nch - 1);
        put_o();
        __builtin_amdgcn_sched_barrier(0);
        // in the loop's order: its waits cover the loads of both
#pragma unroll
        for (int s = 0; s < NKT; ++s) load_a(nch - 1, s);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tb = 0; tb < NB; ++tb) load_b(nch - 1, tb);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tb = 0; tb < NB; ++tb) load_q(nch - 1, tb);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int tb = 0; tb < NB; ++tb) load_k(nch - 1, tb);
        load_g(nch - 1);
    }
    __syncthreads();
    for (int m = nch - 1; m >= 0; --m) {
        const int c0 = t0 + m * C, L = min(C, t1 - c0);
        const size_t gh = (size_t)(g0 + m) * H + h;
        if (own) {  // dS_out of this chunk
#pragma unroll
            for (int u = 0; u < KPW; ++u)
#pragma unroll
                for (int jt = 0; jt < NJT; ++jt)
                    stv(a.dso + (((gh * NKT + kt0 + u) * NJ + vt * NJT + jt) * 64 + lane) * 4,
                        S[u][jt]);
        }
        // Psi = (A_qk L^-1)^T scale dO + KA dS_out = dV, row block w
        // partial sums by key tile modulo NP, [NP][NJT]
        floatx4 x[NJT], xp[CF::NP * NJT];
#pragma unroll
        for (int i = 0; i < CF::NP * NJT; ++i) xp[i] = zero4();
#pragma unroll
        for (int s = 0; s < NKT; s += CF::NP) {
            floatx4 av[CF::NP * NJT], bv[CF::NP * NJT];
#pragma unroll
            for (int i = 0; i < CF::NP * NJT; ++i) {
                const int st = s + i / NJT, jt = i % NJT;
                av[i] = ka[st];
                bv[i] = ldv(s_S + (16 * jt + li) * LDK + 16 * st + 4 * lg);
            }
            mmn(xp, av, bv);
#pragma unroll
            for (int i = 0; i < CF::NP; ++i) load_a(m - 1, s + i);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the tiles tb < w are zero (wave 0 has all four): zeros times the wave's own rows of dO, so
        // that a value that is not finite in an earlier row stays out of this block; two partial sums
        floatx4 xo[2 * NJT];
#pragma unroll
        for (int i = 0; i < 2 * NJT; ++i) xo[i] = zero4();
#pragma unroll
        for (int tb = 0; tb < NB; tb += 2) {
            floatx4 av[2 * NJT], bv[2 * NJT];
#pragma unroll
            for (int i = 0; i < 2 * NJT; ++i) {
                const int t = tb + i / NJT, jt = i % NJT;
                av[i] = t >= w ? ba[t] : zero4();
                bv[i] = ldv(s_O + (16 * jt + li) * LDC + 16 * max(t, w) + 4 * lg);
            }
            mmn(xo, av, bv);
            load_b(m - 1, tb);
            load_b(m - 1, tb + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int jt = 0; jt < NJT; ++jt) {
            x[jt] = xo[jt] + xo[NJT + jt] + sum_parts<CF::NP, NJT>(xp + jt);
            stv(s_P + (16 * jt + li) * LDC + 16 * w + 4 * lg, x[jt]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {  // rows past the end of the sequence are not stored
                const int t = 16 * w + 4 * lg + r;
                store_row(rdv, t < L, ((uint32_t)(c0 + t) * H + h) * DV + j0 + 16 * jt + li,
                          x[jt][r]);
            }
        }
        load_o(m - 1);
        // dS_in^T = dS_out^T diag(gamma_C) + (scale dO)^T Qbar - Psi^T Kbar; the dO term needs no
        // other wave's Psi and runs before the barrier
        floatx4 uq[KPW * NJT];
        state_prod(uq, s_O, qb, [&](int tb) { load_q(m - 1, tb); });
        __syncthreads();
        {
            floatx4 up[KPW * NJT];
            state_prod(up, s_P, nk, [&](int tb) { load_k(m - 1, tb); });
#pragma unroll
            for (int u = 0; u < KPW; ++u)
#pragma unroll
                for (int jt = 0; jt < NJT; ++jt)
                    S[u][jt] = fma4(S[u][jt], gc[u], up[u * NJT + jt] + uq[u * NJT + jt]);
            if (own) put_state();
        }
        put_o();
        load_g(m - 1);
        __syncthreads();
    }
    if (a.dS0 && own) {
#pragma unroll
        for (int u = 0; u < KPW; ++u)
#pragma unroll
            for (int jt = 0; jt < NJT; ++jt) stv(a.dS0 + state_at(u, jt), S[u][jt]);
    }
}

// ------------------------------------------------------------------------------------------
// bw_grad: chunk-parallel gradients of the memory scan and the variance-adjoint coefficients
// ------------------------------------------------------------------------------------------
// Wave w of 4 owns row block w: dq, dk and dkappa of its 16 x 16 tiles (one per 16 channels) stay
// in its registers, and the gates, keys and queries of a lane's tokens 4 g .. 4 g + 3 and channel
// are at once the rows of its results and the operands that the other row blocks contract over.
//  0. Delta = L^-1 X to LDS, wave w the value tiles w, w + 4.
//  1. products over the value columns: Psi S_in^T, dO S_in^T and Delta dS_out^T on the owned tiles
//     (state tiles straight from memory: each is fetched again for the next 16 columns as soon as
//     it is used), dO Delta^T and Psi Delta^T (the adjoints of B and T) on the lower 16 x 16 blocks
//     of row block w; sum_j S_in,ij dS_out,ij.
//  2. the terms through T and B, whose entries carry gamma_t / gamma_s per channel, by slabs of
//     two channel tiles. For 16-token blocks b > c the ratio is the decay from the start of block
//     b to t, times that of the blocks between, times that from s to the end of block c, each
//     <= 1. The column side is scaled by the last and staged (kappa to the block's end, q and k
//     from its start; two buffers, so one barrier per slab); the sum over the blocks runs as a
//     Horner scheme in the block decays that starts from the S_in (dS_out) term, and the result
//     is scaled by the first. Inside a diagonal block both sides are referenced to its token 8 (a
//     factor saturates at 2^100, beyond the inverse of any 8-token decay above 2^-100) and stay
//     with the wave.
// The log-decay adjoint of an entry is then q dq + k dk - kappa dkappa; its chunk-end part enters
// through column sums.
// 79 KB of LDS and 256 registers: two workgroups per CU, so that one's loads, barriers and scalar
// phases run under the other's MFMAs. B4 T4096 H16 d128: 696 us against 1222 us with LDS slabs of
// the state and exponentials of float64 log-decays; eight waves with every channel staged at once
// (156 KB, one workgroup per CU) took 1013 us. Its float32 MFMAs take 300 us (41% of the matrix
// cores' cycles); it moves 2.9 GB past the L2, which a copy does in 600 us. The compiler keeps 65
// values per lane in scratch at DK = 128 (264 bytes, 0.28 GB of the writes; isotropic 57 with gates
// per channel, 23 with one per head; none at smaller DK): phase 1 holds p3, p4, p5 (96 registers)
// and a step's state tiles (64) at once, phase 2 the inputs of the tiles ahead.
template <int DK>
struct GradLds {
    static constexpr int NKT = DK / 16, NJM = 8;  // value tiles of 16 columns at most
    static constexpr int SCT = NKT < 2 ? NKT : 2, NS = NKT / SCT;  // tiles of a slab, slabs
    static constexpr size_t SLAB = (size_t)12 * SCT * 1024;  // kappa, q, k operands [3][4][SCT]
    // Delta [4][NJM] tiles (phase 1); then two slab buffers; then the block maps [4][DK]
    static constexpr size_t MAIN = cmax((size_t)4 * NJM * 1024, 2 * SLAB);
    static constexpr size_t OFF_BR = MAIN;                                  // dB [NLT], LDL
    static constexpr size_t OFF_TR = OFF_BR + (size_t)NLT * 16 * LDL * 4;   // dT [NLT], LDL
    static constexpr size_t OFF_SG = OFF_TR + (size_t)NLT * 16 * LDL * 4;  // block decays [4][DK]
    static constexpr size_t OFF_CP = OFF_SG + (size_t)4 * DK * 4;       // column sums [4][DK]
    static constexpr size_t OFF_BT = OFF_CP + (size_t)4 * DK * 4;       // block totals [4][DK]
    static constexpr size_t OFF_P6 = OFF_BT + (size_t)4 * DK * 4;       // [DK]
    static constexpr size_t TOTAL = al16(OFF_P6 + (size_t)DK * 4);
};

template <class TI, int DK, int VARIANT, bool APC>
__global__ __launch_bounds__(NTH) __attribute__((amdgpu_waves_per_eu(2))) void bw_grad(Args a)
{
    using R = BwRec<DK>;
    using LY = GradLds<DK>;
    constexpr bool DIAG = VARIANT == 0;
    constexpr int NKT = DK / 16, SCT = LY::SCT, NS = LY::NS;
    constexpr int NCHAN = DIAG ? DK : 1;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float* s_D = (float*)smem;
    float* s_op = (float*)smem;  // [2][3][4][SCT] tiles
    float* s_br = (float*)(smem + LY::OFF_BR);
    float* s_tr = (float*)(smem + LY::OFF_TR);
    float* s_g = (float*)(smem + LY::OFF_SG);
    float* s_cp = (float*)(smem + LY::OFF_CP);
    float* s_bt = (float*)(smem + LY::OFF_BT);
    float* s_p6 = (float*)(smem + LY::OFF_P6);
    float2* s_bm = (float2*)smem;  // diagonal: block maps [4][DK]
    float* s_ab = (float*)smem;    // isotropic: A, B [2][C]

    const int H = a.H, DV = a.DV, NJ = DV / 16;
    const int g = (int)(blockIdx.x / H), h = (int)(blockIdx.x % H);
    int n, c0, c1;
    bool last;
    if (!locate_chunk<C>(a.cm, g, n, c0, c1, last)) return;
    const int L = c1 - c0;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lg = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t gh = (size_t)g * H + h;
    const float* __restrict__ rec = a.rec + gh * a.recn;
    constexpr uint32_t es = sizeof(TI);
    const rsrc_t rq = make_rsrc(a.q, a.in.bytes_k), rk = make_rsrc(a.k, a.in.bytes_k);
    const rsrc_t ra = make_rsrc(a.alpha, APC || DIAG ? a.in.bytes_k : a.in.bytes_h);
    const rsrc_t rdq = make_rsrc(a.dq, a.bytes_dk);
    const int tr0 = 16 * w + 4 * lg;  // the lane's rows tr0 .. tr0 + 3
    // byte offset of row tr0, channel li of a [.., H, DK] input, of a per-head one; per row
    const uint32_t ok0 = (((uint32_t)(c0 + tr0) * H + h) * DK + li) * es, okr = (uint32_t)H * DK * es;
    const uint32_t oh0 = ((uint32_t)(c0 + tr0) * H + h) * es, ohr = (uint32_t)H * es;
    typedef typename Raw1<TI>::type RV;
    auto raw_alpha = [&](int r, int ct) {
        if constexpr (DIAG || APC) return Raw1<TI>::load(ra, ok0 + r * okr + 16 * ct * es);
        else return Raw1<TI>::load(ra, oh0 + r * ohr);
    };
    auto raw_k = [&](int r, int ct) { return Raw1<TI>::load(rk, ok0 + r * okr + 16 * ct * es); };
    auto raw_q = [&](int r, int ct) { return Raw1<TI>::load(rq, ok0 + r * okr + 16 * ct * es); };
    // rows past the end of the sequence: no decay, zero key and query
    auto in_row = [&](RV x, int r, float pad) {
        return tr0 + r < L ? Raw1<TI>::f32(x) : pad;
    };

    // ---- 0. Delta ------------------------------------------------------------------------------
    {
        const float* xt = a.xt + gh * C * DV + 4 * lane;
        for (int ks = w; ks < NJ; ks += 4) {  // Delta^T = X^T L^-T
            floatx4 xf[NB];
#pragma unroll
            for (int sb = 0; sb < NB; ++sb) xf[sb] = ldv(xt + (sb * NJ + ks) * 256);
#pragma unroll
            for (int tb = 0; tb < NB; ++tb) {
                floatx4 acc = zero4();
#pragma unroll
                for (int sb = 0; sb <= tb; ++sb)
                    acc += mm(zero4(), xf[sb], ldv(rec + R::LI + ltile(tb, sb) * 256 + 4 * lane));
                stv(s_D + ((tb * NJ + ks) * 64 + lane) * 4, acc);
            }
        }
    }
    // ---- 1. products over the value columns --------------------------------------------------
    typedef TI TO __attribute__((ext_vector_type(4)));
    const bool rowok = 16 * w + li < L, dook = rowok && a.dO;
    const size_t orow = ((size_t)(c0 + min(16 * w + li, L - 1)) * H + h) * DV + 4 * lg;
    const float* pp = a.dv + orow;
    const TI* po = (const TI*)(a.dO ? a.dO : a.v) + orow;  // always a valid row
    auto psi = [&](floatx4 x) {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = rowok ? x[e] : 0.f;
        return x;
    };
    auto dout = [&](TO x) {
        floatx4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = dook ? (float)x[e] : 0.f;
        return y;
    };
    floatx4 sv[NKT], gv[NKT];
    const float* ps = a.ckpt + gh * DK * DV + 4 * lane;
    const float* pg = a.dso + gh * DK * DV + 4 * lane;
#pragma unroll
    for (int k = 0; k < NKT; ++k) {
        sv[k] = ldv(ps + (size_t)k * NJ * 256);
        gv[k] = ldv(pg + (size_t)k * NJ * 256);
    }
    floatx4 pv = ldv(pp);
    TO ov = *reinterpret_cast<const TO*>(po);
    __syncthreads();
    // the adjoints of B and T: dB = scale dO Delta^T (s <= t), dT = -Psi Delta^T (s < t); each
    // 16-column product is summed from zero, then added (shorter chains of roundings). Only the
    // wave itself reads its row block by rows, the later blocks' waves by columns
    {
        floatx4 p1[NB], p2[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) p1[b] = p2[b] = zero4();
        for (int ks = 0; ks < NJ; ++ks) {
            const int kn = ks + 1 < NJ ? ks + 1 : 0;
            const floatx4 aP = psi(pv), aO = dout(ov);
            pv = ldv(pp + 16 * kn);
            ov = *reinterpret_cast<const TO*>(po + 16 * kn);
#pragma unroll
            for (int sb = 0; sb < NB; ++sb)
                if (sb <= w) {
                    const floatx4 bD = ldv(s_D + ((sb * NJ + ks) * 64 + lane) * 4);
                    floatx4 t2[2] = {zero4(), zero4()};
                    mmn(t2, {aO, aP}, {bD, bD});
                    p1[sb] += t2[0];
                    p2[sb] += t2[1];
                }
        }
#pragma unroll
        for (int sb = 0; sb < NB; ++sb)
            if (sb <= w) {
                const int o = ltile(w, sb) * 16 * LDL + 4 * lg * LDL + li;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s_br[o + r * LDL] = sb < w || li <= 4 * lg + r ? a.scale * p1[sb][r] : 0.f;
                    s_tr[o + r * LDL] = sb < w || li < 4 * lg + r ? -p2[sb][r] : 0.f;
                }
            }
    }
    floatx4 p3[NKT], p4[NKT], p5[NKT];
#pragma unroll
    for (int k = 0; k < NKT; ++k) p3[k] = p4[k] = p5[k] = zero4();
    {
        float p6 = 0.f, p6b = 0.f;  // wave w: channel tiles w, w + 4; the lane's channel and columns
#pragma unroll 1
        for (int ks = 0; ks < NJ; ++ks) {
            const int kn = min(ks + 1, NJ - 1);
            const floatx4 aP = psi(pv), aO = dout(ov);
            pv = ldv(pp + 16 * kn);
            ov = *reinterpret_cast<const TO*>(po + 16 * kn);
            const floatx4 aD = ldv(s_D + ((w * NJ + ks) * 64 + lane) * 4);
#pragma unroll
            for (int k = 0; k < NKT; ++k) {
                const floatx4 x = sv[k], y = gv[k];
                // (without a branch: one here splits the loop and its registers)
                const float s = fmaf(x[3], y[3], fmaf(x[2], y[2], fmaf(x[1], y[1], x[0] * y[0])));
                (k < 4 ? p6 : p6b) += (k & 3) == w ? s : 0.f;
                floatx4 t3[3] = {zero4(), zero4(), zero4()};
                mmn(t3, {aP, aO, aD}, {x, x, y});
                p3[k] += t3[0];
                p4[k] += t3[1];
                p5[k] += t3[2];
                sv[k] = ldv(ps + (size_t)(k * NJ + kn) * 256);
                gv[k] = ldv(pg + (size_t)(k * NJ + kn) * 256);
            }
        }
        p6 += __shfl_xor(p6, 16, 64);
        p6 += __shfl_xor(p6, 32, 64);
        if (lg == 0 && w < NKT) s_p6[16 * w + li] = p6;
        if constexpr (NKT > 4) {
            p6b += __shfl_xor(p6b, 16, 64);
            p6b += __shfl_xor(p6b, 32, 64);
            if (lg == 0) s_p6[16 * (w + 4) + li] = p6b;
        }
    }
    auto by_rows = [&](const float* m, int tl) { return ldv(m + tl * 16 * LDL + li * LDL + 4 * lg); };
    auto by_cols = [&](const float* m, int tl) {
        const float* p = m + tl * 16 * LDL + 4 * lg * LDL + li;
        return floatx4{p[0], p[LDL], p[2 * LDL], p[3 * LDL]};
    };
    const floatx4 dnv = ldv(rec + R::DEN + tr0);  // gain denominators of the lane's rows
    floatx4 idn, btv = zero4();                   // diagonal: their inverses; isotropic: beta
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        idn[r] = 1.f / dnv[r];
        if constexpr (!DIAG) btv[r] = rec[R::PH + tr0 + r] / dnv[r];
    }
    auto phat_at = [&](int ct) {
        return DIAG ? ldv(rec + R::PH + ((size_t)(w * NKT + ct) * 64 + lane) * 4) : zero4();
    };
    struct Raw {
        RV al[4], k[4], q[4];
        floatx4 ph;
    };
    Raw in[SCT];
    auto load2 = [&](int ct0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < SCT; ++u) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                in[u].al[r] = raw_alpha(r, ct0 + u);
                in[u].k[r] = raw_k(r, ct0 + u);
                in[u].q[r] = raw_q(r, ct0 + u);
            }
            in[u].ph = phat_at(ct0 + u);
        }
    };
    load2(0);
    __syncthreads();  // Delta is dead: the slab buffers over it

    // ---- 2. terms through T and B; per slab the gradients of its tiles are then complete: dq out,
    // dk and dkappa kept in p3 and p5, the log-decay adjoint q dq + k dk - kappa dkappa in p4 as
    // its suffix sums over the block (alpha dalpha = sum over t >= s; the chunk-end terms enter at
    // the last token) ---------------------------------------------------------------------------
    float rp0[4] = {0.f, 0.f, 0.f, 0.f}, rp1[4] = {0.f, 0.f, 0.f, 0.f};
    float rp2[4] = {0.f, 0.f, 0.f, 0.f};
    const int dt = ltile(w, w);
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
        float* s_ke = s_op + (sl & 1) * (LY::SLAB / 4);
        float* s_qs = s_ke + 4 * SCT * 256;
        float* s_ks = s_qs + 4 * SCT * 256;
        floatx4 gq[SCT], gk[SCT], gp[SCT];  // the diagonal block's terms, then the gradients
        floatx4 asv[SCT], bev[SCT];         // decay from the block's start, to its end
        floatx4 kx[SCT], qx[SCT], kp[SCT];
#pragma unroll
        for (int u = 0; u < SCT; ++u) {
            const int ct = SCT * sl + u;
            floatx4 al;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                al[r] = in_row(in[u].al[r], r, 1.f);
                kx[u][r] = in_row(in[u].k[r], r, 0.f);
                qx[u][r] = in_row(in[u].q[r], r, 0.f);
                kp[u][r] = DIAG ? in[u].ph[r] * kx[u][r] * idn[r] : btv[r] * kx[u][r];
                if constexpr (!DIAG) {
                    rp1[r] = fmaf(kx[u][r], kx[u][r], rp1[r]);
                    if (APC) rp2[r] = fmaf(al[r], al[r], rp2[r]);
                }
            }
            // inclusive products from the lane's first row and exclusive ones to its last; the
            // other lane groups' totals
            floatx4 pre, suf;
            pre[0] = al[0];
            pre[1] = pre[0] * al[1];
            pre[2] = pre[1] * al[2];
            pre[3] = pre[2] * al[3];
            suf[3] = 1.f;
            suf[2] = al[3];
            suf[1] = suf[2] * al[2];
            suf[0] = suf[1] * al[1];
            const float g0 = __shfl(pre[3], li, 64), g1 = __shfl(pre[3], li + 16, 64);
            const float g2 = __shfl(pre[3], li + 32, 64), g3 = __shfl(pre[3], li + 48, 64);
            const float before = (lg > 0 ? g0 : 1.f) * (lg > 1 ? g1 : 1.f) * (lg > 2 ? g2 : 1.f);
            const float after = (lg < 3 ? g3 : 1.f) * (lg < 2 ? g2 : 1.f) * (lg < 1 ? g1 : 1.f);
            if (lg == 0) s_g[w * DK + 16 * ct + li] = (g0 * g1) * (g2 * g3);
            // referenced to token 8: rows from 8 on by the decay since, earlier ones by the
            // inverse of the decay up to it; kappa by the reciprocal factors
            const float mid = lg == 0 ? g1 : (lg == 3 ? g2 : 1.f);
            floatx4 km, qm, pm, amd, bmd, ke, qs, ks;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float f = (lg < 2 ? suf[r] : pre[r]) * mid, fi = inv_decay(f);
                amd[r] = lg < 2 ? fi : f;
                bmd[r] = lg < 2 ? f : fi;
                asv[u][r] = before * pre[r];
                bev[u][r] = after * suf[r];
                km[r] = amd[r] * kx[u][r];
                qm[r] = amd[r] * qx[u][r];
                pm[r] = bmd[r] * kp[u][r];
                ke[r] = bev[u][r] * kp[u][r];
                qs[r] = asv[u][r] * qx[u][r];
                ks[r] = asv[u][r] * kx[u][r];
            }
            const int o = ((w * SCT + u) * 64 + lane) * 4;
            stv(s_ke + o, ke);
            stv(s_qs + o, qs);
            stv(s_ks + o, ks);
            gq[u] = mm(zero4(), by_rows(s_br, dt), pm) * amd;
            gk[u] = mm(zero4(), by_rows(s_tr, dt), pm) * amd;
            gp[u] = mm(mm(zero4(), by_cols(s_br, dt), qm), by_cols(s_tr, dt), km) * bmd;
        }
        if (sl + 1 < NS) load2(SCT * (sl + 1));
        __syncthreads();
#pragma unroll
        for (int u = 0; u < SCT; ++u) {
            const int ct = SCT * sl + u;
            const int i = 16 * ct + li;
            float gb[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) gb[b] = s_g[b * DK + i];
            // rows of block w as the later token: the S_in term, then the earlier blocks
            floatx4 oB = p4[ct] * a.scale, oT = -p3[ct];
#pragma unroll
            for (int jb = 0; jb < 3; ++jb)
                if (jb < w) {
                    const floatx4 bk = ldv(s_ke + ((jb * SCT + u) * 64 + lane) * 4);
                    oB = fma4(oB, gb[jb], mm(zero4(), by_rows(s_br, ltile(w, jb)), bk));
                    oT = fma4(oT, gb[jb], mm(zero4(), by_rows(s_tr, ltile(w, jb)), bk));
                }
            // as the earlier token: the dS_out term, then the later blocks from the last
            floatx4 oP = p5[ct];
            float rest = 1.f;  // decay of the blocks after w
#pragma unroll
            for (int ib = 3; ib > 0; --ib)
                if (ib > w) {
                    const int o = ((ib * SCT + u) * 64 + lane) * 4, tl = ltile(ib, w);
                    const floatx4 t = mm(zero4(), by_cols(s_br, tl), ldv(s_qs + o)) +
                                      mm(zero4(), by_cols(s_tr, tl), ldv(s_ks + o));
                    oP = fma4(oP, gb[ib], t);
                    rest *= gb[ib];
                }
            gq[u] = fma4(oB, asv[u], gq[u]);
            gk[u] = fma4(oT, asv[u], gk[u]);
            gp[u] = fma4(oP, bev[u], gp[u]);
            // the tail operand's part of dkappa, for the chunk-end decay
            const floatx4 tl = p5[ct] * bev[u] * rest;
            float cs = 0.f;
            floatx4 suf;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                store_row(rdq, tr0 + r < L, ((uint32_t)(c0 + tr0 + r) * H + h) * DK + i, gq[u][r]);
                cs = fmaf(kp[u][r], tl[r], cs);
                suf[r] = qx[u][r] * gq[u][r] + kx[u][r] * gk[u][r] - kp[u][r] * gp[u][r];
                rp0[r] = fmaf(gp[u][r], DIAG ? kp[u][r] : kx[u][r], rp0[r]);
            }
            cs += __shfl_xor(cs, 16, 64);
            cs += __shfl_xor(cs, 32, 64);
            if (lg == 0) s_cp[w * DK + i] = cs;
            // suffix within the tile: the lane's rows, then the lanes of the later rows
#pragma unroll
            for (int r = 2; r >= 0; --r) suf[r] += suf[r + 1];
            const float g1 = __shfl(suf[0], li + 16, 64), g2 = __shfl(suf[0], li + 32, 64);
            const float g3 = __shfl(suf[0], li + 48, 64);
            suf += (lg < 1 ? g1 : 0.f) + (lg < 2 ? g2 : 0.f) + (lg < 3 ? g3 : 0.f);
            if (lg == 0) s_bt[w * DK + i] = suf[0];
            p4[ct] = suf;
            p3[ct] = gk[u];
            p5[ct] = gp[u];
        }
    }
    // row sums over the channels (diagonal: the gain denominator's adjoint; isotropic: dbeta,
    // ||k||^2, sum alpha^2)
    float irr[4], rrv[4], ddv[4];  // 1 / r, r and (diagonal) the denominators' adjoint
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        rp0[r] = row16_sum(rp0[r]);
        if constexpr (!DIAG) {
            rp1[r] = row16_sum(rp1[r]);
            if (APC) rp2[r] = row16_sum(rp2[r]);
        }
        ddv[r] = -rp0[r] * idn[r];
        rrv[r] = tr0 + r < L ? ld<TI>(a.r, (size_t)(c0 + tr0 + r) * H + h) : 1.f;
        irr[r] = __builtin_amdgcn_rcpf(rrv[r]);
    }
    __syncthreads();

    // ---- dalpha's log-decay part, dk without the variance adjoint, and the coefficients of the
    // variance adjoint lambda_{t-1} = A_t lambda_t + B_t ----------------------------------------
#pragma unroll
    for (int ct = 0; ct < NKT; ++ct) {
        const int i = 16 * ct + li;
        const size_t o = gh * C * DK + ((size_t)(w * NKT + ct) * 64 + lane) * 4;
        const floatx4 ph = phat_at(ct);
        float off = rec[R::GC + i] * s_p6[i];
#pragma unroll
        for (int b = 0; b < 4; ++b) off += s_cp[b * DK + i] + (b > w ? s_bt[b * DK + i] : 0.f);
        floatx4 kx, al, dal, dkp;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            al[r] = in_row(raw_alpha(r, ct), r, 1.f);
            kx[r] = DIAG ? in_row(raw_k(r, ct), r, 0.f) : 0.f;
            dal[r] = tr0 + r < L ? (p4[ct][r] + off) * __builtin_amdgcn_rcpf(al[r]) : 0.f;
            if constexpr (DIAG)  // through kappa's numerator and its denominator
                dkp[r] = p3[ct][r] + (p5[ct][r] * idn[r] + 2.f * ddv[r] * kx[r]) * ph[r];
            else
                dkp[r] = fmaf(btv[r], p5[ct][r], p3[ct][r]);
        }
        stv(a.dal + o, dal);
        stv(a.dkp + o, dkp);
        if constexpr (DIAG) {
            floatx4 cv;
            float mx = 1.f, my = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                cv[r] = tr0 + r < L ? (p5[ct][r] * idn[r] + ddv[r] * kx[r]) * kx[r] : 0.f;
            stv(a.bcf + o, cv);
            // the block's map of the variance adjoint (lambda_start = mx lambda_end + my): the
            // lane's rows composed from the last down, then the lane groups in time order
            // (f o g: x -> f.x (g.x x + g.y) + f.y)
#pragma unroll
            for (int r = 3; r >= 0; --r) {
                const float a2 = al[r] * al[r];
                const float ig = __builtin_amdgcn_rcpf(fmaf(a.mu * kx[r] * kx[r] * irr[r], ph[r],
                                                            1.f));
                const float av = a2 * ig * ig, bv = a2 * cv[r];
                mx *= av;
                my = fmaf(av, my, bv);
            }
            float px = __shfl(mx, lane + 16, 64), py = __shfl(my, lane + 16, 64);
            my = fmaf(mx, py, my);  // groups 0, 2: own rows after the next group's
            mx *= px;
            px = __shfl(mx, lane + 32, 64);
            py = __shfl(my, lane + 32, 64);
            my = fmaf(mx, py, my);  // group 0: rows 0-7 after rows 8-15
            mx *= px;
            if (lg == 0) s_bm[w * DK + i] = make_float2(mx, my);
        }
    }
    if (li == 0)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int t = tr0 + r;
            if constexpr (DIAG) {
                a.aux[gh * C + t] = ddv[r];
            } else {  // one value per token
                const bool ok = t < L;
                const float rr = rrv[r], dn = dnv[r], dbeta = rp0[r], nk = rp1[r];
                const float al = in_row(raw_alpha(r, 0), r, 1.f);
                const float aa = APC ? rp2[r] / (float)DK : al * al;
                const float u = a.mu * nk / ((float)DK * rr), gg = 1.f + u * rec[R::PH + t];
                const float av = ok ? aa / (gg * gg) : 1.f;
                const float bv = ok ? aa * dbeta * rr / (dn * dn) : 0.f;
                a.acf[gh * C + t] = av;
                a.bcf[gh * C + t] = bv;
                a.aux[gh * 2 * C + t] = dbeta;
                a.aux[gh * 2 * C + C + t] = nk;
                s_ab[t] = av;
                s_ab[C + t] = bv;
            }
        }
    // the chunk's map of the variance adjoint from its end to its start, per channel:
    // lambda_start = m.x lambda_end + m.y, the steps lambda_{t-1} = A_t lambda_t + B_t composed
    // from the last token down: diagonal, the four row blocks' maps in time order; isotropic,
    // the one chain's coefficients
    __syncthreads();
    if constexpr (DIAG) {
        if (tid < DK) {
            float2 m = s_bm[3 * DK + tid];
#pragma unroll
            for (int b = 2; b >= 0; --b) {
                const float2 f = s_bm[b * DK + tid];
                m = make_float2(f.x * m.x, fmaf(f.x, m.y, f.y));
            }
            a.cmap[gh * NCHAN + tid] = m;
        }
    } else if (tid == 0) {
        float mx = 1.f, my = 0.f;
#pragma unroll 16
        for (int t = C - 1; t >= 0; --t) {
            mx *= s_ab[t];
            my = fmaf(s_ab[t], my, s_ab[C + t]);
        }
        a.cmap[gh * NCHAN] = make_float2(mx, my);
    }
}

// ------------------------------------------------------------------------------------------
// bw_scan: the variance adjoint backwards over the chunks, one thread per (sequence, head,
// channel): each chunk's composed map (from bw_grad) applied in reverse; the adjoint at every
// chunk's end is kept for bw_final, which replays the chunk's tokens from it
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void bw_scan(Args a, int nchan)
{
    const int gid = (int)(blockIdx.x * 64 + threadIdx.x);
    const int H = a.H;
    if (gid >= a.cm.N * H * nchan) return;
    const int slot = gid / nchan, c = gid % nchan, n = slot / H, h = slot % H;
    int t0, t1, g0, nch;
    seq_span(a.cm, n, t0, t1);
    seq_chunks<C>(a.cm, n, t0, t1, g0, nch);
    float lp = a.dP_T ? a.dP_T[(size_t)slot * nchan + c] : 0.f;
    for (int cb = nch; cb > 0; cb -= 16) {  // chunks cb - 1 down to max(cb - 16, 0)
        float2 mv[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int ci = max(cb - 1 - e, 0);
            mv[e] = a.cmap[((size_t)(g0 + ci) * H + h) * nchan + c];
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int ci = cb - 1 - e;
            if (ci >= 0) {
                a.lpe[((size_t)(g0 + ci) * H + h) * nchan + c] = lp;
                lp = fmaf(mv[e].x, lp, mv[e].y);
            }
        }
    }
    if (a.dP0) a.dP0[(size_t)slot * nchan + c] = lp;
}

// ------------------------------------------------------------------------------------------
// bw_final: token-local gradients of the gain stage. One wave per (block of 16 tokens, 64
// channels), lane = channel: a lane holds its channel's tokens, and every tile, input and gradient
// row is one contiguous access per wave. Diagonal: the chunk's adjoint lambda enters at its last
// token; the blocks' maps are composed in LDS, then each block replays its tokens. Bound by HBM:
// 160 KB in, 96 KB out per (chunk, head) at DK = 128 in bf16: 205 us at B4 T4096 H16 (5.1 TB/s)
// against 288 us with row-major partial gradients updated in place (384 KB).
// ------------------------------------------------------------------------------------------
template <int DK>
struct FinalCfg {
    static constexpr int NCH = (DK + 63) / 64;  // waves per block
    static constexpr int NT = 64 * NB * NCH;
};

template <class TI, int DK, int VARIANT, bool APC>
__global__ __launch_bounds__((FinalCfg<DK>::NT)) void bw_final(Args a)
{
    using R = BwRec<DK>;
    using CF = FinalCfg<DK>;
    constexpr bool DIAG = VARIANT == 0;
    constexpr int NCHAN = DIAG ? DK : 1, NKT = DK / 16, NCH = CF::NCH;
    __shared__ float2 s_bm[DIAG ? NB * DK : 1];
    __shared__ float s_pe[DIAG ? NB * DK : 1];
    __shared__ float s_r[C], s_sum[NCH][C];
    __shared__ float s_av[C], s_bv[C], s_lp[C], s_dnk[C], s_da[C];  // isotropic
    const int H = a.H;
    const int g = (int)(blockIdx.x / H), h = (int)(blockIdx.x % H);
    int n, c0, c1;
    bool last;
    if (!locate_chunk<C>(a.cm, g, n, c0, c1, last)) return;
    const int L = c1 - c0;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int b = w / NCH, hf = w % NCH, i = min(64 * hf + lane, DK - 1);
    const bool act = 64 * hf + lane < DK;
    const size_t gh = (size_t)g * H + h;
    const float* __restrict__ rec = a.rec + gh * a.recn;
    const int Lw = L - SL * b;  // tokens of this block in the sequence (may be <= 0)
    constexpr uint32_t es = sizeof(TI);
    const rsrc_t rk = make_rsrc(a.k, a.in.bytes_k);
    const rsrc_t ra = make_rsrc(a.alpha, APC || DIAG ? a.in.bytes_k : a.in.bytes_h);
    const uint32_t row0 = (uint32_t)(c0 + SL * b) * H + h;
    // a tile array by columns: the lane's tokens 4 e .. + 3 of the block
    const size_t po = ((size_t)(b * NKT + (i >> 4)) * 64 + (i & 15)) * 4;
    auto cols = [&](const float* p, int e) { return ldv(p + po + 64 * e); };
    typename Raw1<TI>::type kraw[SL], araw[SL];
#pragma unroll
    for (int j = 0; j < SL; ++j) {
        const uint32_t rw = row0 + (uint32_t)(j * H);
        kraw[j] = Raw1<TI>::load(rk, (rw * DK + i) * es);
        araw[j] = Raw1<TI>::load(ra, (APC || DIAG ? rw * DK + i : rw) * es);
    }
    floatx4 dl[4], dp[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        dl[e] = cols(a.dal + gh * C * DK, e);
        dp[e] = cols(a.dkp + gh * C * DK, e);
    }
    if (tid < C) s_r[tid] = tid < L ? ld<TI>(a.r, (size_t)(c0 + tid) * H + h) : 1.f;
    if constexpr (DIAG) {
        floatx4 ph[4], cv[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            ph[e] = cols(rec + R::PH, e);
            cv[e] = cols(a.bcf + gh * C * DK, e);
        }
        const float lend = a.lpe[gh * NCHAN + i];
        const float pp0 = rec[R::PP_D + i];
        __syncthreads();
        float kx[SL], ax[SL], ig[SL];  // keys, gates, 1 / (1 + u p_hat) (hardware reciprocals)
        float mx = 1.f, my = 0.f;
#pragma unroll
        for (int j = SL - 1; j >= 0; --j) {
            const bool ok = j < Lw;
            kx[j] = ok ? Raw1<TI>::f32(kraw[j]) : 0.f;
            ax[j] = ok ? Raw1<TI>::f32(araw[j]) : 1.f;
            const float u = a.mu * kx[j] * kx[j] * __builtin_amdgcn_rcpf(s_r[SL * b + j]);
            ig[j] = __builtin_amdgcn_rcpf(fmaf(u, ph[j >> 2][j & 3], 1.f));
            const float a2 = ax[j] * ax[j], av = a2 * ig[j] * ig[j];
            mx *= av;
            my = fmaf(av, my, a2 * cv[j >> 2][j & 3]);
        }
        if (act) {
            s_bm[b * DK + i] = make_float2(mx, my);
            s_pe[b * DK + i] = ph[3][3] * ig[SL - 1];  // p after the block
        }
        __syncthreads();
        float lp = lend;
#pragma unroll
        for (int bb = NB - 1; bb > 0; --bb)
            if (bb > b) {
                const float2 m = s_bm[bb * DK + i];
                lp = fmaf(m.x, lp, m.y);
            }
        const float pin = b == 0 ? pp0 : s_pe[(b - 1) * DK + i];  // p before the block
#pragma unroll
        for (int j = SL - 1; j >= 0; --j) {
            const float ir = __builtin_amdgcn_rcpf(s_r[SL * b + j]);
            const float p = ph[j >> 2][j & 3], ig2 = ig[j] * ig[j];
            const float dph = fmaf(lp, ig2, cv[j >> 2][j & 3]);
            const float du = -lp * p * p * ig2;
            const float pp = j > 0 ? ph[(j - 1) >> 2][(j - 1) & 3] * ig[j > 0 ? j - 1 : 0] : pin;
            const float s2 = wave_sum(act ? du * kx[j] * kx[j] : 0.f);
            if (lane == 0) s_sum[hf][SL * b + j] = s2;
            if (j < Lw && act) {
                const size_t o = ((size_t)row0 + (size_t)j * H) * DK + i;
                a.dk[o] = dp[j >> 2][j & 3] + 2.f * du * a.mu * kx[j] * ir;
                a.dalpha[o] = dl[j >> 2][j & 3] + dph * 2.f * ax[j] * pp;
                a.domega[o] = dph;
            }
            lp = ax[j] * ax[j] * dph;
        }
        __syncthreads();
        if (tid < L) {
            float s2 = 0.f;
#pragma unroll
            for (int u = 0; u < NCH; ++u) s2 += s_sum[u][tid];
            const float ir = __builtin_amdgcn_rcpf(s_r[tid]);
            a.dr[(size_t)(c0 + tid) * H + h] = a.aux[gh * C + tid] - s2 * a.mu * ir * ir;
        }
    } else {
        if (tid < C) {
            s_av[tid] = a.acf[gh * C + tid];
            s_bv[tid] = a.bcf[gh * C + tid];
        }
        if (!APC) {  // the gate's log-decay part: one gate per head and token
#pragma unroll
            for (int j = 0; j < SL; ++j) {
                const float sd = wave_sum(act ? dl[j >> 2][j & 3] : 0.f);
                if (lane == 0) s_sum[hf][SL * b + j] = sd;
            }
        }
        __syncthreads();
        if (tid == 0) {  // lambda_{t-1} = A_t lambda_t + B_t from the chunk's end
            float lp = a.lpe[gh];
#pragma unroll 16
            for (int t = C - 1; t >= 0; --t) {
                s_lp[t] = lp;
                lp = fmaf(s_av[t], lp, s_bv[t]);
            }
        }
        __syncthreads();
        if (tid < C) {
            const int t = tid;
            const float rr = s_r[t], dn = rec[R::DEN + t], bh = rec[R::PH + t];
            const float pp = rec[R::PP_I + t], lp = s_lp[t];
            const float dbeta = a.aux[gh * 2 * C + t], nk = a.aux[gh * 2 * C + C + t];
            const float u = a.mu * nk / ((float)DK * rr), gg = 1.f + u * bh, ig2 = 1.f / (gg * gg);
            const float dbh = lp * ig2 + dbeta * rr / (dn * dn);
            const float du = -lp * bh * bh * ig2;
            const float da = dbh * pp;
            s_dnk[t] = -dbeta * bh * bh / (dn * dn) + du * a.mu / ((float)DK * rr);
            s_da[t] = da;
            if (t < L) {
                const size_t row = (size_t)(c0 + t) * H + h;
                a.dr[row] = -dbeta * bh / (dn * dn) - du * a.mu * nk / ((float)DK * rr * rr);
                a.domega[row] = dbh;
                if (!APC) {
                    float sd = 0.f;
#pragma unroll
                    for (int v = 0; v < NCH; ++v) sd += s_sum[v][t];
                    a.dalpha[row] = sd + da * 2.f * ld<TI>(a.alpha, row);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < SL; ++j)
            if (j < Lw && act) {
                const int t = SL * b + j;
                const size_t o = ((size_t)row0 + (size_t)j * H) * DK + i;
                a.dk[o] = dp[j >> 2][j & 3] + 2.f * Raw1<TI>::f32(kraw[j]) * s_dnk[t];
                if (APC)
                    a.dalpha[o] = dl[j >> 2][j & 3] +
                                  s_da[t] * 2.f * Raw1<TI>::f32(araw[j]) * (1.f / (float)DK);
            }
    }
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
size_t rec_floats(int dk, bool diag)
{
    switch (dk) {
    case 16: return BwRec<16>::size(diag);
    case 32: return BwRec<32>::size(diag);
    case 64: return BwRec<64>::size(diag);
    default: return BwRec<128>::size(diag);
    }
}

template <class TI, int DK, int NJT>
hipError_t run_walks(const Args& a, hipStream_t st)
{
    const size_t nh8 = ((size_t)a.cm.N * a.H + 7) / 8 * 8;
    const dim3 grid((unsigned)(nh8 * (size_t)(a.DV / (16 * NJT))));
    hipLaunchKernelGGL((bw_fwalk<TI, DK, NJT>), grid, dim3(NTH), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((bw_rwalk<TI, DK, NJT>), grid, dim3(NTH), 0, st, a);
    return hipGetLastError();
}

template <class TI, int DK, int VARIANT, bool APC>
hipError_t run(const BwdCall& bc, hipStream_t st)
{
    using VC = fwd::VarCfg<TI, DK, VARIANT, APC>;
    using PC = PrepCfg<TI, DK, VARIANT, APC>;
    const SeqArgs& sa = bc.sa;
    const bool packed = sa.cu_seqlens != nullptr;
    const size_t recn = BwRec<DK>::size(VARIANT == 0);
    const BwMap m = bw_map(VARIANT, packed, sa.N, sa.B, sa.T, sa.H, DK, bc.dv, recn);
    char* ws = (char*)bc.workspace;
    hipError_t e;
    ChunkMap cm;
    cm.cu = sa.cu_seqlens;
    cm.choff = packed ? (const int32_t*)(ws + m.choff) : nullptr;
    cm.N = sa.N;
    cm.T = sa.T;
    cm.ntok = sa.B * sa.T;
    cm.maxch = m.maxch;
    if (packed &&
        (e = launch_chunk_table(sa.cu_seqlens, sa.N, cm.ntok, C, m.maxch,
                                (int32_t*)(ws + m.choff), st)) != hipSuccess)
        return e;
    const size_t ntok = (size_t)sa.B * sa.T * sa.H;
    fwd::InArgs in = {};
    in.q = bc.q; in.k = bc.k; in.alpha = bc.alpha; in.omega = bc.omega; in.r = bc.r;
    in.bytes_k = (uint32_t)(ntok * DK * sizeof(TI));
    in.bytes_h = (uint32_t)(ntok * sizeof(TI));
    in.H = sa.H;
    in.mu = bc.mu;
    float4* summ = (float4*)(ws + m.summ);
    float2* carry = (float2*)(ws + m.carry);
    const dim3 cgrid((unsigned)((size_t)m.maxch * sa.H));
    if (m.maxch > 0) {
        hipLaunchKernelGGL((fwd::summary_kernel<TI, VC>), cgrid, dim3(fwd::NTH), 0, st, in, cm,
                           summ);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = launch_carry_scan(summ, bc.P0, cm, C, sa.H, VC::NCHAN, carry, nullptr, st)) !=
            hipSuccess)
            return e;
    }
    Args a = {};
    a.q = bc.q; a.k = bc.k; a.v = bc.v; a.alpha = bc.alpha; a.omega = bc.omega; a.r = bc.r;
    a.dO = bc.dO; a.S0 = bc.S0; a.dS_T = bc.dS_T; a.dP_T = bc.dP_T;
    a.dq = bc.gq; a.dk = bc.gk; a.dv = bc.gv; a.dalpha = bc.galpha; a.domega = bc.gomega;
    a.dr = bc.gr; a.dS0 = bc.gS0; a.dP0 = bc.gP0;
    a.in = in;
    a.cm = cm;
    a.H = sa.H;
    a.DV = bc.dv;
    a.bytes_v = (uint32_t)(ntok * bc.dv * sizeof(TI));
    // below 4 GiB: the inputs are below 2 GiB in either type
    a.bytes_dv = (uint32_t)(ntok * bc.dv * 4);
    a.bytes_dk = (uint32_t)(ntok * DK * 4);
    a.mu = bc.mu;
    a.scale = bc.scale;
    a.carry = carry;
    a.rec = (float*)(ws + m.rec);
    a.recn = recn;
    a.ckpt = (float*)(ws + m.ckpt);
    a.xt = (float*)(ws + m.xt);
    a.dso = (float*)(ws + m.dso);
    a.dkp = (float*)(ws + m.dkp);
    a.dal = (float*)(ws + m.dal);
    a.bcf = (float*)(ws + m.bcf);
    a.acf = (float*)(ws + m.acf);
    a.aux = (float*)(ws + m.aux);
    a.cmap = (float2*)(ws + m.cmap);
    a.lpe = (float*)(ws + m.lpe);
    if ((e = fwd::set_lds(bw_prep<TI, PC>, PC::TOTAL)) != hipSuccess ||
        (e = fwd::set_lds(bw_grad<TI, DK, VARIANT, APC>, GradLds<DK>::TOTAL)) != hipSuccess)
        return e;
    if (m.maxch > 0) {
        hipLaunchKernelGGL((bw_prep<TI, PC>), cgrid, dim3(NTH), PC::TOTAL, st, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    e = bc.dv < 32 ? run_walks<TI, DK, 1>(a, st) : run_walks<TI, DK, 2>(a, st);
    if (e != hipSuccess) return e;
    if (m.maxch > 0) {
        hipLaunchKernelGGL((bw_grad<TI, DK, VARIANT, APC>), cgrid, dim3(NTH), GradLds<DK>::TOTAL,
                           st, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const int nthr = sa.N * sa.H * VC::NCHAN;
    hipLaunchKernelGGL(bw_scan, dim3((unsigned)((nthr + 63) / 64)), dim3(64), 0, st, a,
                       (int)VC::NCHAN);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (m.maxch > 0) {
        hipLaunchKernelGGL((bw_final<TI, DK, VARIANT, APC>), cgrid, dim3(FinalCfg<DK>::NT), 0, st,
                           a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

template <class TI, int DK>
hipError_t run_v(const BwdCall& bc, hipStream_t st)
{
    if (bc.variant == 0) return run<TI, DK, 0, true>(bc, st);
    if (bc.apc) return run<TI, DK, 1, true>(bc, st);
    return run<TI, DK, 1, false>(bc, st);
}

template <class TI>
hipError_t run_dk(const BwdCall& bc, hipStream_t st)
{
    switch (bc.dk) {
    case 16: return run_v<TI, 16>(bc, st);
    case 32: return run_v<TI, 32>(bc, st);
    case 64: return run_v<TI, 64>(bc, st);
    case 128: return run_v<TI, 128>(bc, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace bwd

size_t backward_workspace_bytes(int variant, bool packed, int N, int B, int T, int H, int dk,
                                int dv)
{
    return bwd::bw_map(variant, packed, N, B, T, H, dk, dv, bwd::rec_floats(dk, variant == 0)).total;
}

hipError_t launch_backward(const BwdCall& bc, hipStream_t stream)
{
    if (bc.dtype == KDN_F32) return bwd::run_dk<float>(bc, stream);
    return bwd::run_dk<bf16>(bc, stream);
}

}  // namespace kdn
