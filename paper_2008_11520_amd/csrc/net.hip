// Per-patch GRU (Eq. (gru), no biases) and MLP head on gfx950 matrix cores.
//
//   z  = sigma(W_z x + U_z h)          r = sigma(W_r x + U_r h)
//   h' = z h + (1 - z) tanh(W_h x + U_h (r h))
//   d  = M2 relu(M1 h')   (or M h')
//
// Patches are the rows of tall-skinny products.  A workgroup takes tiles of 16, 32
// or 64 patch rows (the batch table counts row tiles of 64); its waves own hidden
// tiles of 16 units and run the whole chain on 16 x 16 MFMA tiles with FP32 accumulation:
//   phase 1: [x | h] against the stacked gate weights [W_g | U_g] (U_h part 0),
//   gates in registers, r*h to LDS,
//   phase 2: (r*h) against U_h, then the update of h (FP32 state),
//   MLP: h' -> LDS -> M1 -> relu -> LDS -> M2 -> per-patch output.
// Operands are FP32 (v_mfma_f32_16x16x4_f32) or BF16 with round-to-nearest-
// even (v_mfma_f32_16x16x32_bf16).  Weights are pre-packed at create time
// into per-lane fragments so that each lane reads 16 contiguous bytes.
//
// Fragment convention (both forms): in k-chunk kc, lane l = i + 16 q holds
// operand values at k = kc*KC + q*KQ + e, e < KQ (A: row i; B: column i).
// The 16 x 16 f32 result tile gives lane l rows 4 q + e (e < 4) of column i.
#include "device.h"
#include "fp8.h"
#include "internal.h"
#include "net_index.h"

namespace dnnmg {


template <int PREC> struct Op;

// FP32 operands: a 16-wide k-chunk is four 16x16x4 MFMAs; lane element e of
// the chunk feeds the e-th of them.
template <> struct Op<0> {
    typedef float T;
    typedef f4 Frag;
    static constexpr int KC = 16, KQ = 4;
    __device__ static inline f4 mma(f4 acc, Frag a, Frag b)
    {
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, acc, 0, 0, 0);
        return acc;
    }
    __device__ static inline T cvt(float x) { return x; }
};

// BF16 operands: one 16x16x32 MFMA per 32-wide k-chunk.
template <> struct Op<1> {
    typedef __bf16 T;
    typedef bf8 Frag;
    static constexpr int KC = 32, KQ = 8;
    __device__ static inline f4 mma(f4 acc, Frag a, Frag b)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
    }
    __device__ static inline T cvt(float x) { return (__bf16)x; }
};


// Streamed kernel: FP32 operands, and the BF16 shapes that the persistent
// kernels below do not cover (H = 32 or 96 at K = 3; the reset after U_h at H = 128
// or K = 3; an MLP width other than 0 or H) or are slower for (H >= 96 on few
// patches, see launch_net).
//
// A workgroup takes R = 64 patches (16 where there are few: the products of one
// row tile follow each other on one matrix core, so a grid that does not fill
// the chip is timed by them).  Wave w owns hidden tile w % HT for RT of the
// row tiles, so the workgroup reads each weight fragment once from L2 (twice
// at H = 32) and every fragment feeds RT row tiles.  The operand rows
// [x | h | 0] lie in LDS at a pitch of an odd number of 16-byte pieces (the 16
// rows of a fragment read fall in distinct banks); once the gate products are
// done the same bytes hold r * h, h' and the MLP hidden layer.  Products are
// formed transposed (weights x activations^T), so that lane (li, lq) holds patch
// row 16 rt + li and the four units ucol = 16 ht + 4 lq .. + 3: the state is read once,
// in that layout (the operand and the update share it), and state, r * h, h' and
// outputs move as vectors.  The gate fragments of the next AHEAD k-chunks are
// requested before a chunk's products.  The k-chunks that hold the state alone
// skip the candidate gate, whose weights there are zero (164 of 180 products of a
// row tile and hidden tile at K = 2, H = Hm = 64).
// FP32 is bound by the matrix cores: 656 products of 32 cycles per 16 patches at
// that shape, 140 us for 1024 x 256 patches at 2.4 GHz (164 us at the 134 TFLOP/s
// that a register-only loop of this instruction reaches); 286 -> 204 us against
// wave pairs that read every weight fragment twice and the rows from global
// memory inside the k-loop.  Eight waves of two row tiles measured slower (232 us).
struct StreamRows {
    int lda, bytes;   // row pitch in elements, and LDS bytes of the tile
};
template <int PREC, int H, int R>
__host__ __device__ inline StreamRows stream_rows(int kc1, int Hm)
{
    typedef Op<PREC> O;
    constexpr int V = 16 / (int)sizeof(typename O::T);
    StreamRows r;
    const int w = kc1 * O::KC;
    r.lda = (w / V) % 2 ? w : w + V;
    const int ldh = H + V, ldm = Hm > 0 ? Hm + V : 0;
    const int tail = ldh + (ldh > ldm ? ldh : ldm);      // h', then r * h and the MLP hidden layer
    r.bytes = R * (r.lda > tail ? r.lda : tail) * (int)sizeof(typename O::T);
    return r;
}

// Waves of a workgroup: one per hidden tile, at least four; at H = 96 two per
// hidden tile (six waves would load the four SIMDs unevenly: 300 x 200 patches,
// K = 2, FP32 step 159.8 -> 140.1 us), and registers for two workgroups per CU.
constexpr int kFewRows = 16;   // patches of a workgroup where there are few (see launch_net_t)
template <int H, int R> constexpr int stream_waves() { return R < 64 ? H / 16 * (R / 16) : (H == 96 ? 12 : (H / 16 < 4 ? 4 : H / 16)); }
template <int H, int R> constexpr int stream_simd_waves() { return H == 96 && R == 64 ? 6 : 2; }

template <int PREC, int H, int R>
__device__ __forceinline__ void stream_tile(const FlowArgs &f, int blk, const NetArgs &net, unsigned char *lds)
{
    typedef Op<PREC> O;
    typedef typename O::T T;
    typedef typename O::Frag Frag;
    constexpr int KC = O::KC, KQ = O::KQ, HC = H / KC, V = 16 / (int)sizeof(T);
    constexpr int HT = H / 16, NW = stream_waves<H, R>(), NT = 64 * NW, RT = R / 16 * HT / NW;
    // k-chunks requested ahead: a chunk's products take 4 times as long in FP32,
    // and one row tile's a quarter of four's
    constexpr int AHEAD = R < 64 ? 4 : (PREC == 0 ? 1 : 2);
    constexpr int LDH = H + V;
    typedef T T4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(1))) float gfloat;
    typedef __attribute__((address_space(1))) f4 gf4;
    typedef float v2 __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(1))) v2 gv2;

    const int P = f.nx * f.ny;
    const int nin = net.nin, nout = net.nout, Hm = net.Hm, kc1 = net.kc1;
    const bool reset_after = net.reset_after != 0;
    const int lda = stream_rows<PREC, H, R>(kc1, Hm).lda, ldm = Hm + V;
    const int tid = tile_thread();
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int li = lane & 15, lq = lane >> 4;
    const int ht = wave % HT, rt0 = RT * (wave / HT);
    const int ucol = 16 * ht + 4 * lq;
    const int row0 = blk * R, nrows = min(R, P - row0);

    T *const sA = reinterpret_cast<T *>(lds);          // [x | h | 0]
    T *const sHp = sA, *const sR = sA + R * LDH, *const sAm = sR;
    const gptr<Frag> B1 = pinned<Frag>(net.B1);
    const gptr<Frag> B2 = pinned<Frag>(net.B2);
    const gptr<Frag> B3 = pinned<Frag>(net.B3);
    const gptr<Frag> B4 = pinned<Frag>(net.B4);
    gfloat *const hG = (gfloat *)(f.h + (size_t)row0 * H);
    gfloat *const dG = (gfloat *)(f.dpatch + (size_t)row0 * nout);

    // ---- the tile's rows to LDS.  x: consecutive 16-byte pieces of memory
    //      (unconditional loads: those past the mesh's last row read its
    //      last piece, and such rows' results are never stored); h: in the
    //      lanes' own layout.
    {
        typedef unsigned int u4 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(1))) const u4 gu4;
        gu4 *const X = (gu4 *)(reinterpret_cast<const T *>(f.X) + (size_t)row0 * nin);
        const unsigned pr = (unsigned)nin / V, np = R * pr, in = (unsigned)nrows * pr;   // pieces per row, per tile, inside
        const unsigned inv = ((1u << 24) + pr - 1) / pr;      // c / pr = c inv >> 24 (c < 64 pr, pr < 128: exact)
        constexpr int U = PREC == 0 ? 7 : 4;
        for (unsigned c0 = tid; c0 < np; c0 += U * NT) {
            u4 x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = X[tile_piece_last(c0 + u * NT, in)];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned c = c0 + u * NT, r = c * inv >> 24;
                if (c < np) *reinterpret_cast<u4 *>(&sA[r * lda + V * (c - r * pr)]) = x[u];
            }
        }
    }
    f4 hold[RT];
#pragma unroll
    for (int q = 0; q < RT; ++q) {
        const int r = 16 * (rt0 + q) + li;
        hold[q] = *(gf4 *)(hG + tile_row(r, nrows) * H + ucol);
    }
    Frag w[AHEAD][3];
    const int kcx = (nin + KC - 1) / KC;            // chunks with input columns
    auto fetch = [&](int kc, Frag (&d)[3]) {
        const int k = min(kc, kc1 - 1);
        d[0] = B1[((0 * HT + ht) * kc1 + k) * 64 + lane];
        d[1] = B1[((1 * HT + ht) * kc1 + k) * 64 + lane];
        d[2] = B1[((2 * HT + ht) * kc1 + min(k, kcx - 1)) * 64 + lane];
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) fetch(i, w[i]);
#pragma unroll
    for (int q = 0; q < RT; ++q) {
        const int r = 16 * (rt0 + q) + li;
        T4 hb;
#pragma unroll
        for (int e = 0; e < 4; ++e) hb[e] = O::cvt(hold[q][e]);
        *reinterpret_cast<T4 *>(&sA[r * lda + nin + ucol]) = hb;
    }
    for (int z = nin + H + 4 * (tid & 3); z < kc1 * KC; z += 16)       // the k-padding
        for (int r = tid >> 2; r < R; r += NT / 4) *reinterpret_cast<T4 *>(&sA[r * lda + z]) = T4{};
    __syncthreads();

    // ---- phase 1: [x | h] against [W_g | U_g], g = z, r, h (U_h comes in phase 2)
    f4 az[RT], ar[RT], ah[RT];
#pragma unroll
    for (int q = 0; q < RT; ++q) az[q] = ar[q] = ah[q] = f4{0.f, 0.f, 0.f, 0.f};
    const T *const arow = sA + (16 * rt0 + li) * lda + lq * KQ;
    auto chunk = [&](int kc, bool cand) {
        Frag nw[3];
        fetch(kc + AHEAD, nw);
        __builtin_amdgcn_sched_barrier(0);   // (the loads stay ahead of the products)
#pragma unroll
        for (int q = 0; q < RT; ++q) {
            const Frag a = *reinterpret_cast<const Frag *>(&arow[16 * q * lda + kc * KC]);
            az[q] = O::mma(az[q], w[0][0], a);
            ar[q] = O::mma(ar[q], w[0][1], a);
            if (cand) ah[q] = O::mma(ah[q], w[0][2], a);
        }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
#pragma unroll
            for (int g = 0; g < 3; ++g) w[i][g] = i + 1 < AHEAD ? w[i + 1][g] : nw[g];
    };
#pragma unroll 1
    for (int kc = 0; kc < kcx; ++kc) chunk(kc, true);
#pragma unroll 1
    for (int kc = kcx; kc < kc1; ++kc) chunk(kc, false);
    Frag w2[HC];
#pragma unroll
    for (int kc = 0; kc < HC; ++kc) w2[kc] = B2[(ht * HC + kc) * 64 + lane];
    __syncthreads();   // every wave is done with the operand rows

    // ---- gates; r*h to LDS (reset after U_h: h itself, r kept for the candidate)
#pragma unroll
    for (int q = 0; q < RT; ++q) {
        const int r = 16 * (rt0 + q) + li;
        T4 rh;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // (BF16 weights come pre-multiplied for 2^x, see sigmoid_l2)
            az[q][e] = PREC == 1 ? sigmoid_l2(az[q][e]) : sigmoid(az[q][e]);
            ar[q][e] = PREC == 1 ? sigmoid_l2(ar[q][e]) : sigmoid(ar[q][e]);
            rh[e] = O::cvt(reset_after ? hold[q][e] : ar[q][e] * hold[q][e]);
        }
        *reinterpret_cast<T4 *>(&sR[r * LDH + ucol]) = rh;
    }
    __syncthreads();

    // ---- phase 2: U_h (r*h) (or U_h h, then times r); new state
    f4 au[RT];
#pragma unroll
    for (int q = 0; q < RT; ++q) au[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < HC; ++kc)
#pragma unroll
        for (int q = 0; q < RT; ++q)
            au[q] = O::mma(au[q], w2[kc], *reinterpret_cast<const Frag *>(&sR[(16 * (rt0 + q) + li) * LDH + kc * KC + lq * KQ]));
#pragma unroll
    for (int q = 0; q < RT; ++q) {
        const int r = 16 * (rt0 + q) + li;
        f4 hn;
        T4 hb;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float z = az[q][e];
            const float u = reset_after ? ar[q][e] * au[q][e] : au[q][e];
            const float hh = PREC == 1 ? tanh_l2(ah[q][e] + u) : fast_tanh(ah[q][e] + u);
            hn[e] = hh + z * (hold[q][e] - hh);   // z h + (1 - z) hh
            hb[e] = O::cvt(hn[e]);
        }
        if (r < nrows) *(gf4 *)(hG + r * H + ucol) = hn;
        *reinterpret_cast<T4 *>(&sHp[r * LDH + ucol]) = hb;
    }
    __syncthreads();

    // ---- MLP head; the wave takes hidden and output tiles ht, ht + HT, ...
    auto product = [&](f4 (&acc)[RT], const T *src, int ld, int kcn, gptr<Frag> Bw, int tile) {
#pragma unroll
        for (int q = 0; q < RT; ++q) acc[q] = f4{0.f, 0.f, 0.f, 0.f};
        Frag wk = Bw[(tile * kcn) * 64 + lane];
        for (int kc = 0; kc < kcn; ++kc) {
            const Frag wn = Bw[(tile * kcn + min(kc + 1, kcn - 1)) * 64 + lane];
#pragma unroll
            for (int q = 0; q < RT; ++q)
                acc[q] = O::mma(acc[q], wk, *reinterpret_cast<const Frag *>(&src[(16 * (rt0 + q) + li) * ld + kc * KC + lq * KQ]));
            wk = wn;
        }
    };
    const int ot_n = (nout + 15) / 16;
    f4 acc[RT];
    if (Hm > 0) {
        for (int mt = ht; mt < Hm / 16; mt += HT) {
            product(acc, sHp, LDH, HC, B3, mt);
#pragma unroll
            for (int q = 0; q < RT; ++q) {
                T4 m;
#pragma unroll
                for (int e = 0; e < 4; ++e) m[e] = O::cvt(fmaxf(acc[q][e], 0.f));
                *reinterpret_cast<T4 *>(&sAm[(16 * (rt0 + q) + li) * ldm + 16 * mt + 4 * lq]) = m;
            }
        }
        __syncthreads();
    }
    for (int ot = ht; ot < ot_n; ot += HT) {
        if (Hm > 0) product(acc, sAm, ldm, Hm / KC, B4, ot);
        else product(acc, sHp, LDH, HC, B3, ot);
        const int oc = 16 * ot + 4 * lq;
#pragma unroll
        for (int q = 0; q < RT; ++q) {
            const int r = 16 * (rt0 + q) + li;
            // nout is even: the pairs (oc, oc+1), (oc+2, oc+3) are inside or outside together
            if (r < nrows) {
                gfloat *o = dG + r * nout + oc;
                if (oc < nout) *(gv2 *)o = v2{acc[q][0], acc[q][1]};
                if (oc + 2 < nout) *(gv2 *)(o + 2) = v2{acc[q][2], acc[q][3]};
            }
        }
    }
}

// Single flow: one tile per block.  Batched: the blocks stride over the
// table's tiles of all flows, so the grid need not match the batch.
template <int PREC, int H, int R, bool BATCHED>
__global__ __launch_bounds__(64 * (stream_waves<H, R>()), (stream_simd_waves<H, R>())) void k_net(FlowArgs single, const BatchTable *__restrict__ bt, NetArgs net)
{
    extern __shared__ __align__(16) unsigned char s_rows[];
    if (!BATCHED) {
        stream_tile<PREC, H, R>(single, blockIdx.x, net, s_rows);
        return;
    }
    const int total = bt->prefix[kKindNet][bt->nflows];
#pragma unroll 1
    for (int g = blockIdx.x; g < total; g += gridDim.x) {
        int blk = g;
        const FlowArgs &f = *batch_flow(bt, kKindNet, blk);
        stream_tile<PREC, H, R>(f, blk, net, s_rows);
        __syncthreads();   // LDS is reused by the next tile
    }
}


// ---------------------------------------------------------------- FP8 E4M3
// Every product takes E4M3 operands with one FP32 scale per row and
// accumulates in FP32: weights per output row (packed at create), the
// network input per patch (quantised by the defect kernel), and the state h,
// r*h, h' and the MLP hidden layer per patch, quantised here.  The input and
// the state of the gate products carry separate scales, so their k-chunks are
// accumulated separately: the input part is rescaled by s_x / s_h before the
// state part is added, and the sum by s_h s_w at the end.
typedef long f8x8;   // 8 E4M3 codes: one MFMA operand fragment

__device__ inline f8x8 mma_fp8_operand(const uint8_t *p) { return *reinterpret_cast<const f8x8 *>(p); }

__device__ inline f4 mma_fp8(f4 acc, f8x8 a, f8x8 b)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b, acc, 0, 0, 0);
}

// Row maximum over the 16 lanes that share lq (the 16 columns of a tile).
__device__ inline float max16(float m)
{
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
    return m;
}

template <int H>
__device__ __forceinline__ void net_tile_fp8(const FlowArgs &f, int blk, NetArgs net)
{
    constexpr int KC = 32, KQ = 8, HT = H / 16, HC = H / 32;
    constexpr int LDH = H + 16;                // bytes per staged row (16-byte padding)
    constexpr int LDM = 256 + 16;
    constexpr int MT_MAX = 256 / 16;           // MLP hidden tiles (Hm <= 256)
    __shared__ __align__(16) uint8_t sR[4][16 * LDH];
    __shared__ __align__(16) uint8_t sHp[4][16 * LDH];
    __shared__ __align__(16) uint8_t sAm[4][16 * LDM];

    const int P = f.nx * f.ny;
    const int nin = net.nin, nout = net.nout, Hm = net.Hm, kc1 = net.kc1;
    const int XS = xstride_fp8(nin), kcx = XS / KC;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int li = lane & 15, lq = lane >> 4;
    const int rbase = blk * kNetRows + wave * 16;   // first patch row of this wave
    const int arow = rbase + li;                    // row this lane supplies A values for
    const bool aok = arow < P;
    const uint8_t *X8 = reinterpret_cast<const uint8_t *>(f.X);
    const f8x8 *B1 = reinterpret_cast<const f8x8 *>(net.B1);
    const f8x8 *B2 = reinterpret_cast<const f8x8 *>(net.B2);
    const f8x8 *B3 = reinterpret_cast<const f8x8 *>(net.B3);
    const f8x8 *B4 = reinterpret_cast<const f8x8 *>(net.B4);

    // ---- the state row of this lane's A row: scale and codes
    float hv[HC][KQ];
    float mh = 0.0f;
#pragma unroll
    for (int kh = 0; kh < HC; ++kh)
#pragma unroll
        for (int e = 0; e < KQ; ++e) {
            hv[kh][e] = aok ? f.h[(size_t)arow * H + kh * KC + lq * KQ + e] : 0.0f;
            mh = fmaxf(mh, fabsf(hv[kh][e]));
        }
    mh = fmaxf(mh, __shfl_xor(mh, 16));
    mh = fmaxf(mh, __shfl_xor(mh, 32));
    mh = fmaxf(mh, kFp8MinMax);
    const float rh_li = 448.0f / mh, sh_li = mh / 448.0f;
    f8x8 qh[HC];
#pragma unroll
    for (int kh = 0; kh < HC; ++kh) {
        const uint32_t lo = pack4_e4m3(hv[kh][0] * rh_li, hv[kh][1] * rh_li, hv[kh][2] * rh_li, hv[kh][3] * rh_li);
        const uint32_t hi = pack4_e4m3(hv[kh][4] * rh_li, hv[kh][5] * rh_li, hv[kh][6] * rh_li, hv[kh][7] * rh_li);
        qh[kh] = (f8x8)(((unsigned long)hi << 32) | lo);
    }

    // ---- phase 1, input chunks: x . [W_z W_r W_h]
    f4 az[HT], ar[HT], ah[HT];
#pragma unroll
    for (int t = 0; t < HT; ++t) az[t] = ar[t] = ah[t] = f4{0.f, 0.f, 0.f, 0.f};
    for (int kc = 0; kc < kcx; ++kc) {
        const f8x8 a = aok ? mma_fp8_operand(X8 + (size_t)arow * XS + kc * KC + lq * KQ) : 0;
#pragma unroll
        for (int t = 0; t < HT; ++t) {
            az[t] = mma_fp8(az[t], a, B1[((0 * HT + t) * kc1 + kc) * 64 + lane]);
            ar[t] = mma_fp8(ar[t], a, B1[((1 * HT + t) * kc1 + kc) * 64 + lane]);
            ah[t] = mma_fp8(ah[t], a, B1[((2 * HT + t) * kc1 + kc) * 64 + lane]);
        }
    }
    // accumulator element e is patch row rbase + 4 lq + e
    float sx[4], sh[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int row = rbase + 4 * lq + e;
        sx[e] = row < P ? f.sx[row] : 1.0f;
        sh[e] = __shfl(sh_li, 4 * lq + e);
        const float ratio = sx[e] / sh[e];
#pragma unroll
        for (int t = 0; t < HT; ++t) { az[t][e] *= ratio; ar[t][e] *= ratio; }
    }
    // ---- phase 1, state chunks: h . [U_z U_r] (the candidate has no U block here)
#pragma unroll
    for (int kh = 0; kh < HC; ++kh)
#pragma unroll
        for (int t = 0; t < HT; ++t) {
            az[t] = mma_fp8(az[t], qh[kh], B1[((0 * HT + t) * kc1 + kcx + kh) * 64 + lane]);
            ar[t] = mma_fp8(ar[t], qh[kh], B1[((1 * HT + t) * kc1 + kcx + kh) * 64 + lane]);
        }

    // ---- gates; r*h.  Lane holds rows rbase + 4 lq + e, column 16 t + li.
    float hold[HT][4];
    float mr[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = rbase + 4 * lq + e, k = 16 * t + li;
            const float h0 = row < P ? f.h[(size_t)row * H + k] : 0.f;
            hold[t][e] = h0;
            az[t][e] = sigmoid(az[t][e] * sh[e] * net.s1[k]);
            const float rh = sigmoid(ar[t][e] * sh[e] * net.s1[H + k]) * h0;
            ar[t][e] = rh;
            mr[e] = fmaxf(mr[e], fabsf(rh));
            ah[t][e] *= sx[e] * net.s1[2 * H + k];
        }
    float srh[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float m = fmaxf(max16(mr[e]), kFp8MinMax);
        const float r = 448.0f / m;
        srh[e] = m / 448.0f;
#pragma unroll
        for (int t = 0; t < HT; ++t) sR[wave][(4 * lq + e) * LDH + 16 * t + li] = to_e4m3(ar[t][e] * r);
    }
    __syncthreads();

    // ---- phase 2: (r*h) . U_h^T; new state
    f4 au[HT];
#pragma unroll
    for (int t = 0; t < HT; ++t) au[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < HC; ++kc) {
        const f8x8 a = mma_fp8_operand(&sR[wave][li * LDH + kc * KC + lq * KQ]);
#pragma unroll
        for (int t = 0; t < HT; ++t) au[t] = mma_fp8(au[t], a, B2[(t * HC + kc) * 64 + lane]);
    }
    float mp[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < HT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = rbase + 4 * lq + e, k = 16 * t + li;
            const float z = az[t][e];
            const float hh = fast_tanh(ah[t][e] + au[t][e] * srh[e] * net.s2[k]);
            const float hn = hh + z * (hold[t][e] - hh);   // z h + (1 - z) hh
            if (row < P) f.h[(size_t)row * H + k] = hn;
            au[t][e] = hn;
            mp[e] = fmaxf(mp[e], fabsf(hn));
        }
    float shp[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float m = fmaxf(max16(mp[e]), kFp8MinMax);
        const float r = 448.0f / m;
        shp[e] = m / 448.0f;
#pragma unroll
        for (int t = 0; t < HT; ++t) sHp[wave][(4 * lq + e) * LDH + 16 * t + li] = to_e4m3(au[t][e] * r);
    }
    __syncthreads();

    // ---- MLP head
    const int ot_n = (nout + 15) / 16;
    const uint8_t *src = sHp[wave];
    int lds = LDH, kcs = HC;
    const f8x8 *Bo = B3;
    const float *so = net.s3;
    float sin_[4] = {shp[0], shp[1], shp[2], shp[3]};
    if (Hm > 0) {
        float am[MT_MAX][4];
        float ma[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int mt = 0; mt < MT_MAX; ++mt) {
            if (mt < Hm / 16) {
                f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < HC; ++kc) {
                    const f8x8 a = mma_fp8_operand(&sHp[wave][li * LDH + kc * KC + lq * KQ]);
                    acc = mma_fp8(acc, a, B3[(mt * HC + kc) * 64 + lane]);
                }
                const float sw = net.s3[16 * mt + li];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    am[mt][e] = fmaxf(acc[e] * shp[e] * sw, 0.f);
                    ma[e] = fmaxf(ma[e], am[mt][e]);
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float m = fmaxf(max16(ma[e]), kFp8MinMax);
            const float r = 448.0f / m;
            sin_[e] = m / 448.0f;
#pragma unroll
            for (int mt = 0; mt < MT_MAX; ++mt)
                if (mt < Hm / 16) sAm[wave][(4 * lq + e) * LDM + 16 * mt + li] = to_e4m3(am[mt][e] * r);
        }
        __syncthreads();
        src = sAm[wave];
        lds = LDM;
        kcs = Hm / KC;
        Bo = B4;
        so = net.s4;
    }
    for (int ot = 0; ot < ot_n; ++ot) {
        f4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int kc = 0; kc < kcs; ++kc) {
            const f8x8 a = mma_fp8_operand(&src[li * lds + kc * KC + lq * KQ]);
            acc = mma_fp8(acc, a, Bo[(ot * kcs + kc) * 64 + lane]);
        }
        const int o = 16 * ot + li;
        if (o < nout) {
            const float sw = so[o];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = rbase + 4 * lq + e;
                if (row < P) f.dpatch[(size_t)row * nout + o] = acc[e] * sin_[e] * sw;
            }
        }
    }
}

// Stage entry point: the per-row activation quantiser of the FP8 form on its
// own, one workgroup per row.
__global__ __launch_bounds__(kThreads) void k_quantize(const float *a, int rows, int cols, uint8_t *q, float *s)
{
    __shared__ float sm[kThreads / 64];
    const int row = blockIdx.x;
    const float *ar = a + (size_t)row * cols;
    float m = 0.0f;
    for (int k = threadIdx.x; k < cols; k += kThreads) m = fmaxf(m, fabsf(ar[k]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
    m = fmaxf(m, kFp8MinMax);
    const float r = 448.0f / m;
    if (threadIdx.x == 0) s[row] = m / 448.0f;
    for (int k = threadIdx.x; k < cols; k += kThreads) q[(size_t)row * cols + k] = to_e4m3(ar[k] * r);
}

hipError_t launch_quantize(const float *a, int rows, int cols, uint8_t *q, float *s, hipStream_t st)
{
    hipLaunchKernelGGL(k_quantize, dim3(rows), dim3(kThreads), 0, st, a, rows, cols, q, s);
    return hipGetLastError();
}

template <int H, bool BATCHED>
__global__ __launch_bounds__(kThreads) void k_net_fp8(FlowArgs single, const BatchTable *__restrict__ bt, NetArgs net)
{
    if (!BATCHED) {
        net_tile_fp8<H>(single, blockIdx.x, net);
        return;
    }
    const int total = bt->prefix[kKindNet][bt->nflows];
#pragma unroll 1
    for (int g = blockIdx.x; g < total; g += gridDim.x) {
        int blk = g;
        const FlowArgs &f = *batch_flow(bt, kKindNet, blk);
        net_tile_fp8<H>(f, blk, net);
        __syncthreads();   // LDS is reused by the next tile
    }
}

// Persistent BF16 kernel for K <= 2 and H <= 96 (Hm 0 or H), NIN input columns.
// Two waves per hidden tile: wave w owns hidden tile w % HT for row tiles
// 2 (w / HT) and 2 (w / HT) + 1 of each 64-patch tile, and keeps that hidden
// tile's weight fragments (three gates, U_h) in registers for the whole launch;
// the MLP and output fragments lie in LDS.  The workgroup loops over 64-patch
// row tiles staged through LDS, so each weight fragment is read from memory
// once per workgroup and the loads in flight are the next tiles' rows alone.
// Bound by HBM and the five barriers of a tile: at 1024 x 256 patches and K = 2
// H = 64 takes 56.5 us (241 MB), H = 96 with the paper's input 70 us (308 MB; the
// streamed kernel, which holds two workgroups of six waves per CU and waits for
// its rows at each tile's start, 126 us).  Any spill inside the loop waits for
// the rows in flight (100 us with a second prefetch buffer at H = 96).
template <int H> constexpr int net_reg_threads() { return 8 * H; }

template <int NIN, int H>
__global__ __launch_bounds__(net_reg_threads<H>(), (H == 96 ? 3 : 2)) void k_net_reg(FlowArgs single, const BatchTable *__restrict__ bt,
                                                                                     NetArgs net, int ntiles)
{
    typedef Op<1> O;
    constexpr int NT = net_reg_threads<H>();
    constexpr int KC = 32, KQ = 8, HT = H / 16, HC = H / KC, RTW = 2;
    constexpr int K = NIN == 104 ? 2 : 1, n = 1 << K, nf = (n + 1) * (n + 1), nin = NIN, nout = 2 * nf;
    if (bt) ntiles = bt->prefix[kKindNet][bt->nflows];   // batched: the table's row tiles
    constexpr int KC1 = (nin + H + KC - 1) / KC, KCX = (nin + KC - 1) / KC;   // k-chunks; those with input columns
    // row pitch: an odd number of 16-byte pieces
    constexpr int LDA = (KC1 * KC / 8) % 2 ? KC1 * KC : KC1 * KC + 8;
    constexpr int LDH = H + 8;
    constexpr int OT = (nout + 15) / 16;       // output tiles
    constexpr int WT = HT > OT ? HT : OT;
    constexpr int PADK = KC1 * KC - nin - H;
    static_assert((H == 32 || H == 64 || H == 96) && nin % 8 == 0, "two waves per hidden tile, rows in 16-byte pieces");

    __shared__ __align__(16) __bf16 sA[64 * LDA];
    constexpr int LDS32 = H + 4;              // FP32 state rows, padded against bank conflicts
    __shared__ __align__(16) float sH[64 * LDS32];
    __shared__ __align__(16) __bf16 sR[64 * LDH];
    __shared__ __align__(16) __bf16 sHp[64 * LDH];
    __shared__ __align__(16) __bf16 sAm[64 * LDH];

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int li = lane & 15, lq = lane >> 4;
    const int ht = wave % HT, rt0 = RTW * (wave / HT);
    const int Hm = net.Hm;
    const bool reset_after = net.reset_after != 0;
    const bf8 *B1 = reinterpret_cast<const bf8 *>(net.B1);
    const bf8 *B2 = reinterpret_cast<const bf8 *>(net.B2);
    const bf8 *B3 = reinterpret_cast<const bf8 *>(net.B3);
    const bf8 *B4 = reinterpret_cast<const bf8 *>(net.B4);

    // gate and U_h fragments in registers (the candidate's weights are zero in
    // the chunks of state alone); the MLP fragments in LDS
    __shared__ __align__(16) bf8 sW3[WT * HC * 64];
    __shared__ __align__(16) bf8 sW4[OT * HC * 64];
    constexpr bool W2R = H < 96;               // (at H = 96 U_h lies in LDS too: 12 waves leave 168 registers each)
    __shared__ __align__(16) bf8 sW2[W2R ? 1 : HT * HC * 64];
    bf8 wz[KC1], wr[KC1], wh[KCX], w2[W2R ? HC : 1];
#pragma unroll
    for (int kc = 0; kc < KC1; ++kc) {
        wz[kc] = B1[((0 * HT + ht) * KC1 + kc) * 64 + lane];
        wr[kc] = B1[((1 * HT + ht) * KC1 + kc) * 64 + lane];
    }
#pragma unroll
    for (int kc = 0; kc < KCX; ++kc) wh[kc] = B1[((2 * HT + ht) * KC1 + kc) * 64 + lane];
    if constexpr (W2R) {
#pragma unroll
        for (int kc = 0; kc < HC; ++kc) w2[kc] = B2[(ht * HC + kc) * 64 + lane];
    } else {
        for (int t = tid; t < HT * HC * 64; t += NT) sW2[t] = B2[t];
    }
    const int n3 = (Hm > 0 ? HT : OT) * HC * 64;      // fragments of M1, or of M
    for (int t = tid; t < n3; t += NT) sW3[t] = B3[t];
    if (Hm > 0)
        for (int t = tid; t < OT * HC * 64; t += NT) sW4[t] = B4[t];

    // Tiles are contiguous in memory: the network input (BF16, 64 x nin) and
    // the state (FP32, 64 x H).  Each thread prefetches its 16-byte pieces of
    // the next two tiles into two register buffers while the current one is
    // computed, so two tiles' loads are in flight per workgroup.
    constexpr int XCH = 64 * nin / 8, HCH = 64 * H / 4;            // 16-byte pieces per tile
    constexpr int XPT = (XCH + NT - 1) / NT;
    constexpr int HPT = (HCH + NT - 1) / NT;
    bf8 xrA[XPT], xrB[XPT];
    f4 hrA[HPT], hrB[HPT];
    // A row tile's buffers.  The fields are read in two branches: a pointer
    // that may point at either the kernel argument or the batch table would
    // make them flat loads (and the lambdas below would reach the argument
    // through a generic pointer).
    typedef __attribute__((address_space(1))) float gfloat;
    struct Rows {
        gptr<bf8> X;
        gfloat *h, *dp;
        int nrows;
    };
    const void *const s_X = single.X;
    float *const s_h = single.h, *const s_dp = single.dpatch;
    const int s_P = single.nx * single.ny;
    auto rows_of = [&](int tile) -> Rows {
        int blk = tile;
        const void *X;
        float *h, *dp;
        int P;
        if (bt) {
            const FlowArgs &F = *batch_flow(bt, kKindNet, blk);
            X = F.X; h = F.h; dp = F.dpatch; P = F.nx * F.ny;
        } else {
            X = s_X; h = s_h; dp = s_dp; P = s_P;
        }
        const int row0 = blk * 64;
        Rows r;
        r.X = (gptr<bf8>)(reinterpret_cast<const __bf16 *>(X) + (size_t)row0 * nin);
        r.h = (gfloat *)(h + (size_t)row0 * H);
        r.dp = (gfloat *)(dp + (size_t)row0 * nout);
        r.nrows = min(64, P - row0);
        return r;
    };
    // (index math from tile_thread(): recomputed in each tile instead of
    // hoisted out of the tile loop and held in registers)
    typedef __attribute__((address_space(1))) const f4 gf4;
    auto load_tile = [&](int tile, bf8 (&xr)[XPT], f4 (&hr)[HPT]) {
        const Rows rw = rows_of(tile);
        const int t0 = tile_thread();
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int c = t0 + i * NT;
            xr[i] = tile_piece_in(c, nin / 8, rw.nrows) ? rw.X[c] : bf8{};
        }
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            const int c = t0 + i * NT;
            hr[i] = tile_piece_in(c, H / 4, rw.nrows) ? ((gf4 *)rw.h)[c] : f4{0.f, 0.f, 0.f, 0.f};
        }
    };
    // the k-padding columns of [x | h] stay zero for the whole launch
    if (PADK > 0)
        for (int t = tid; t < 64 * PADK; t += NT) sA[(t / PADK) * LDA + nin + H + t % PADK] = (__bf16)0.f;
    const int G = gridDim.x;
    // (two tiles in flight; one at H = 96, where a second buffer would spill)
    constexpr bool TWO = H < 96;
    if (blockIdx.x < ntiles) load_tile(blockIdx.x, xrA, hrA);
    if (TWO && blockIdx.x + G < ntiles) load_tile(blockIdx.x + G, xrB, hrB);

    // one 64-patch tile: stage the prefetched registers, refill them with
    // tile `next`, compute
    auto process = [&](int tile, bf8 (&xr)[XPT], f4 (&hr)[HPT], int next) {
        const Rows rw = rows_of(tile);
        const int nrows = rw.nrows;
        gfloat *const hg = rw.h;
        gfloat *const dp = rw.dp;

        __syncthreads();   // the previous tile's readers of LDS are done
        const int t1 = tile_thread();
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int c = t1 + i * NT;
            if (c < XCH) *reinterpret_cast<bf8 *>(&sA[(c / (nin / 8)) * LDA + 8 * (c % (nin / 8))]) = xr[i];
        }
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            const int c = t1 + i * NT;
            if (c < HCH) {
                const int r = c / (H / 4), k = 4 * (c % (H / 4));
                *reinterpret_cast<f4 *>(&sH[r * LDS32 + k]) = hr[i];
                bf4 hb;
                hb[0] = (__bf16)hr[i].x; hb[1] = (__bf16)hr[i].y; hb[2] = (__bf16)hr[i].z; hb[3] = (__bf16)hr[i].w;
                *reinterpret_cast<bf4 *>(&sA[r * LDA + nin + k]) = hb;
            }
        }
        if (next < ntiles) load_tile(next, xr, hr);
        __syncthreads();

        // The products are formed transposed (weights x activations^T), so the
        // 16 x 16 result tile gives lane (li, lq) patch row 16 rt + li and the
        // four consecutive hidden units 16 ht + 4 lq + e: gate inputs, r*h, h'
        // and the MLP activations move as 8- and 16-byte vectors.
        const int ucol = 16 * ht + 4 * lq;       // first of this lane's four units
        // ---- phase 1: the three gates of this wave's hidden tile
        f4 az[RTW], ar[RTW], ah[RTW];
#pragma unroll
        for (int q = 0; q < RTW; ++q) az[q] = ar[q] = ah[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < KC1; ++kc)
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const bf8 a = *reinterpret_cast<const bf8 *>(&sA[(16 * (rt0 + q) + li) * LDA + kc * KC + lq * KQ]);
                az[q] = O::mma(az[q], wz[kc], a);
                ar[q] = O::mma(ar[q], wr[kc], a);
                if (kc < KCX) ah[q] = O::mma(ah[q], wh[kc], a);
            }
        f4 hold[RTW];
#pragma unroll
        for (int q = 0; q < RTW; ++q) {
            const int r = 16 * (rt0 + q) + li;
            hold[q] = *reinterpret_cast<const f4 *>(&sH[r * LDS32 + ucol]);
            bf4 rh;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                az[q][e] = sigmoid_l2(az[q][e]);
                ar[q][e] = sigmoid_l2(ar[q][e]);
                // (reset after U_h: h itself, r kept for the candidate)
                rh[e] = (__bf16)(reset_after ? hold[q][e] : ar[q][e] * hold[q][e]);
            }
            *reinterpret_cast<bf4 *>(&sR[r * LDH + ucol]) = rh;
        }
        __syncthreads();

        // ---- phase 2: U_h (r*h); new state
#pragma unroll
        for (int q = 0; q < RTW; ++q) {
            const int r = 16 * (rt0 + q) + li;
            f4 au = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < HC; ++kc) {
                const bf8 a = *reinterpret_cast<const bf8 *>(&sR[r * LDH + kc * KC + lq * KQ]);
                au = O::mma(au, W2R ? w2[W2R ? kc : 0] : sW2[W2R ? 0 : (ht * HC + kc) * 64 + lane], a);
            }
            f4 hn;
            bf4 hb;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float z = az[q][e];
                // h' = z h + (1 - z) c = c + z (h - c), c the candidate state
                const float u = reset_after ? ar[q][e] * au[e] : au[e];
                const float c = tanh_l2(ah[q][e] + u);
                hn[e] = c + z * (hold[q][e] - c);
                hb[e] = (__bf16)hn[e];
            }
            if (r < nrows) *(__attribute__((address_space(1))) f4 *)(hg + r * H + ucol) = hn;
            *reinterpret_cast<bf4 *>(&sHp[r * LDH + ucol]) = hb;
        }
        __syncthreads();

        // ---- MLP head
        const __bf16 *src = sHp;
        if (Hm > 0) {
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const int r = 16 * (rt0 + q) + li;
                f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < HC; ++kc) {
                    const bf8 a = *reinterpret_cast<const bf8 *>(&sHp[r * LDH + kc * KC + lq * KQ]);
                    acc = O::mma(acc, sW3[(ht * HC + kc) * 64 + lane], a);
                }
                bf4 m;
#pragma unroll
                for (int e = 0; e < 4; ++e) m[e] = (__bf16)fmaxf(acc[e], 0.f);
                *reinterpret_cast<bf4 *>(&sAm[r * LDH + ucol]) = m;
            }
            __syncthreads();
            src = sAm;
        }
        for (int ot = ht; ot < OT; ot += HT) {
            const int oc = 16 * ot + 4 * lq;
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const int r = 16 * (rt0 + q) + li;
                f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < HC; ++kc) {
                    const bf8 a = *reinterpret_cast<const bf8 *>(&src[r * LDH + kc * KC + lq * KQ]);
                    acc = O::mma(acc, Hm > 0 ? sW4[(ot * HC + kc) * 64 + lane] : sW3[(ot * HC + kc) * 64 + lane], a);
                }
                // nout is even: the pairs (oc, oc+1), (oc+2, oc+3) are inside or outside together
                if (r < nrows) {
                    typedef float v2 __attribute__((ext_vector_type(2)));
                    typedef __attribute__((address_space(1))) v2 gv2;
                    gfloat *o = dp + r * nout + oc;
                    if (oc < nout) *(gv2 *)o = v2{acc[0], acc[1]};
                    if (oc + 2 < nout) *(gv2 *)(o + 2) = v2{acc[2], acc[3]};
                }
            }
        }
    };
    if constexpr (TWO) {
        for (int tile = blockIdx.x; tile < ntiles; tile += 2 * G) {
            process(tile, xrA, hrA, tile + 2 * G);
            if (tile + G < ntiles) process(tile + G, xrB, hrB, tile + 3 * G);
        }
    } else {
        for (int tile = blockIdx.x; tile < ntiles; tile += G) process(tile, xrA, hrA, tile + G);
    }
}

// Maximum over a group of lanes: the value of lane ^ 16, lane ^ 32 (swaps of
// rows of 16 and of halves, which the vector unit does without LDS) ...
__device__ inline float max_xor16(float m)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float max_xor32(float m)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// ... and over a row of 16 lanes: quads by permutation, then the mirrored half rows and rows.
template <int CTRL>
__device__ inline float max_dpp(float m)
{
    return fmaxf(m, __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(m), CTRL, 0xF, 0xF, true)));
}
__device__ inline float max_row16(float m)
{
    return max_dpp<0x140>(max_dpp<0x141>(max_dpp<0x4E>(max_dpp<0xB1>(m))));
}

// Persistent FP8 kernel (H = 64 or 128, Hm = 0 or H, K <= 3) on tiles of 32
// patches.  One wave per hidden tile: it computes that tile for the tile's two
// row tiles and keeps its gate and U_h fragments in registers for the whole
// launch (90 VGPRs at K = 3, H = 128: the FP8 weights that BF16 could not keep
// resident); the MLP fragments and the per-unit weight scales live in LDS.
// Products are formed transposed (weights x activations^T) as in k_net_reg, so
// a lane holds one patch row and four consecutive units; the per-patch row
// maxima of the quantised activations are reduced over lanes and then over the
// waves of the row through LDS.
// Bound by the chain of a tile, seven barriers and six divisions per row, and
// by the vector unit (830 instructions per wave and tile, as many as the
// memory leaves time for): so the waves that wait for each other are few (four
// at H = 64) and four workgroups of them share a CU.  At 1024 x 256 patches,
// K = 2, H = 64: 70 us, 220 MB at 3.1 TB/s; with one workgroup of eight waves and
// 64 patches per CU 92 us, with two of them 71.5 (113 with its registers
// spilled: per-lane values are derived again in each tile, the state is read
// twice).  On 50 x 30 patches at H = 128 the step went from 33.9 to 26.5 us.
constexpr int kQ8Rows = 32;
template <int H> constexpr int q8p_threads() { return 4 * H; }
// Waves per SIMD that the registers allow: the resident weights take 22 to 48
// VGPRs at K = 1 and 2, up to 90 at K = 3.
constexpr int q8p_waves(int K) { return K <= 2 ? 4 : 2; }

template <int K, int H, int HM>
__global__ __launch_bounds__(q8p_threads<H>(), q8p_waves(K)) void k_net_q8p(FlowArgs single, const BatchTable *__restrict__ bt,
                                                               NetArgs net, int ntiles)
{
    constexpr int n = 1 << K, nf = (n + 1) * (n + 1), nin = 4 * nf + 4, nout = 2 * nf;
    constexpr int KC = 32, KQ = 8;
    constexpr int XS = xstride_fp8(nin), KCX = XS / KC, HC = H / KC, KC1 = KCX + HC;
    constexpr int NT = q8p_threads<H>(), R = kQ8Rows;
    constexpr int HT = H / 16, RTW = R / 16;             // wave w: hidden tile w of all the tile's rows
    constexpr int OT = (nout + 15) / 16;
    constexpr int MC = HM / KC;
    constexpr int LDX = XS + 16, LDQ = H + 16, LDS32 = H + 4;
    constexpr int W3N = (HM > 0 ? HM / 16 : OT) * HC * 64, W4N = HM > 0 ? OT * MC * 64 : 1;
    static_assert(HM == 0 || HM == H, "MLP hidden tiles follow the hidden tiles");
    if (bt) ntiles = bt->prefix[kKindNet][bt->nflows];   // batched: the table's row tiles
    ntiles *= 64 / R;                                    // this kernel's tiles

    __shared__ __align__(16) uint8_t sX[R * LDX];       // network input codes of the tile
    __shared__ __align__(16) float sH[R * LDS32];       // FP32 state of the tile
    __shared__ __align__(16) uint8_t sQ[R * LDQ];       // state codes, then r*h codes
    __shared__ __align__(16) uint8_t sHp[R * LDQ];      // h' codes
    __shared__ __align__(16) uint8_t sAm[R * LDQ];      // MLP hidden codes
    __shared__ __align__(16) f8x8 sW3[W3N];
    __shared__ __align__(16) f8x8 sW4[W4N];
    __shared__ float sMax[HT * R];                     // per-wave partial row maxima
    __shared__ __align__(16) float sRow[4 * R];          // row scales of x and h, their quotient
    constexpr int SO = 3 * H + H + HM;                  // first output scale
    __shared__ __align__(16) float sS[SO + 16 * OT];

    const int tid = threadIdx.x, ht = __builtin_amdgcn_readfirstlane(tid >> 6), lane0 = tid & 63;
    const f8x8 *B1 = reinterpret_cast<const f8x8 *>(net.B1);
    const f8x8 *B2 = reinterpret_cast<const f8x8 *>(net.B2);
    const f8x8 *B3 = reinterpret_cast<const f8x8 *>(net.B3);
    const f8x8 *B4 = reinterpret_cast<const f8x8 *>(net.B4);

    constexpr bool W2R = !(H == 128 && K == 2);          // U_h in registers (there it would spill), or in LDS
    __shared__ __align__(16) f8x8 sW2[W2R ? 1 : HT * HC * 64];
    f8x8 wz[KC1], wr[KC1], wh[KCX], w2[W2R ? HC : 1];
#pragma unroll
    for (int kc = 0; kc < KC1; ++kc) {
        wz[kc] = B1[((0 * HT + ht) * KC1 + kc) * 64 + lane0];
        wr[kc] = B1[((1 * HT + ht) * KC1 + kc) * 64 + lane0];
    }
#pragma unroll
    for (int kc = 0; kc < KCX; ++kc) wh[kc] = B1[((2 * HT + ht) * KC1 + kc) * 64 + lane0];
    if constexpr (W2R) {
#pragma unroll
        for (int kc = 0; kc < HC; ++kc) w2[kc] = B2[(ht * HC + kc) * 64 + lane0];
    } else {
        for (int t = tid; t < HT * HC * 64; t += NT) sW2[t] = B2[t];
    }
    for (int t = tid; t < W3N; t += NT) sW3[t] = B3[t];
    for (int t = tid; t < W4N; t += NT) sW4[t] = HM > 0 ? B4[t] : 0;
    // per-unit weight scales: z | r | candidate | U_h | M1 (or the output's) | output
    for (int t = tid; t < 3 * H; t += NT) sS[t] = net.s1[t];
    for (int t = tid; t < H; t += NT) sS[3 * H + t] = net.s2[t];
    if (HM > 0)
        for (int t = tid; t < H; t += NT) sS[4 * H + t] = net.s3[t];
    for (int t = tid; t < 16 * OT; t += NT)
        sS[SO + t] = t < nout ? (HM > 0 ? net.s4 : net.s3)[t] : 0.0f;
    auto scales = [&](int at) { return *reinterpret_cast<const f4 *>(&sS[at]); };

    // A row tile's buffers.  The fields are read in two branches: a pointer
    // that may point at either the kernel argument or the batch table would
    // make them flat loads (and the lambdas below would reach the argument
    // through a generic pointer).
    typedef __attribute__((address_space(1))) float gfloat;
    struct Rows {
        gptr<uint8_t> X;
        gptr<float> sx;
        gfloat *h, *dp;
        int nrows;
    };
    const void *const s_X = single.X;
    const float *const s_sx = single.sx;
    float *const s_h = single.h, *const s_dp = single.dpatch;
    const int s_P = single.nx * single.ny;
    auto rows_of = [&](int tile) -> Rows {
        int blk = tile / (64 / R);
        const void *X;
        const float *sxp;
        float *h, *dp;
        int P;
        if (bt) {
            const FlowArgs &F = *batch_flow(bt, kKindNet, blk);
            X = F.X; sxp = F.sx; h = F.h; dp = F.dpatch; P = F.nx * F.ny;
        } else {
            X = s_X; sxp = s_sx; h = s_h; dp = s_dp; P = s_P;
        }
        const int row0 = blk * 64 + R * (tile % (64 / R));
        Rows r;
        r.X = (gptr<uint8_t>)(reinterpret_cast<const uint8_t *>(X) + (size_t)row0 * XS);
        r.sx = (gptr<float>)(sxp + row0);
        r.h = (gfloat *)(h + (size_t)row0 * H);
        r.dp = (gfloat *)(dp + (size_t)row0 * nout);
        r.nrows = min(R, P - row0);
        return r;
    };

    // next-tile prefetch into registers: network input codes, FP32 state, x
    // scales (index math from tile_thread(): recomputed in each tile instead
    // of hoisted out of the tile loop and held in registers)
    constexpr int XCH = R * XS / 16, HCH = R * H / 4;
    constexpr int XPT = (XCH + NT - 1) / NT;
    constexpr int HPT = (HCH + NT - 1) / NT;
    typedef unsigned int u4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(1))) const u4 gu4;
    typedef __attribute__((address_space(1))) const f4 gf4;
    u4 xr[XPT];
    f4 hr[HPT];
    float sxr[HPT];                                     // x scale of the row of each state piece
    auto load_tile = [&](int tile) {
        const Rows rw = rows_of(tile);
        const int t0 = tile_thread();
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int c = t0 + i * NT;
            xr[i] = tile_piece_in(c, XS / 16, rw.nrows) ? ((gu4 *)rw.X)[c] : u4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            const int c = t0 + i * NT;
            hr[i] = tile_piece_in(c, H / 4, rw.nrows) ? ((gf4 *)rw.h)[c] : f4{0.f, 0.f, 0.f, 0.f};
            sxr[i] = tile_piece_in(c, H / 4, rw.nrows) ? rw.sx[c / (H / 4)] : 1.0f;
        }
    };
    if (blockIdx.x < ntiles) load_tile(blockIdx.x);

    // row maximum of |v| over the 16 units a wave holds for its row, then over
    // the HT waves of the row (the caller brackets this with barriers)
    auto wave_max = [&](float m, int row, int lq) {
        m = max_xor32(max_xor16(m));
        if (lq == 0) sMax[ht * R + row] = m;
    };
    auto row_max = [&](int row) {
        float m = kFp8MinMax;
#pragma unroll
        for (int t = 0; t < HT; ++t) m = fmaxf(m, sMax[t * R + row]);
        return m;
    };

    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const Rows rw = rows_of(tile);
        const int nrows = rw.nrows;
        gfloat *const hg = rw.h;
        gfloat *const dp = rw.dp;

        // (the rows staged here were last read before the previous tile's later barriers)
        const int t1 = tile_thread();
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int c = t1 + i * NT;
            if (c < XCH) *reinterpret_cast<u4 *>(&sX[(c / (XS / 16)) * LDX + 16 * (c % (XS / 16))]) = xr[i];
        }
        // the state: FP32 rows and their codes; the H / 4 consecutive threads
        // that hold one row's pieces reduce its maximum by shuffles
        static_assert(HCH % NT == 0 && (H / 4) <= 64, "whole rows per pass");
#pragma unroll
        for (int i = 0; i < HPT; ++i) {
            const int c = t1 + i * NT;
            const int row = c / (H / 4), k = 4 * (c % (H / 4));
            *reinterpret_cast<f4 *>(&sH[row * LDS32 + k]) = hr[i];
            float m = fmaxf(fmaxf(fabsf(hr[i].x), fabsf(hr[i].y)), fmaxf(fabsf(hr[i].z), fabsf(hr[i].w)));
            m = max_row16(m);
            if constexpr (H == 128) m = max_xor16(m);
            m = fmaxf(m, kFp8MinMax);
            const float r = 448.0f / m;
            if (k == 0) {
                const float sh = m / 448.0f;
                *reinterpret_cast<f4 *>(&sRow[4 * row]) = f4{sxr[i], sh, sxr[i] / sh, 0.f};
            }
            *reinterpret_cast<uint32_t *>(&sQ[row * LDQ + k]) =
                pack4_e4m3(hr[i].x * r, hr[i].y * r, hr[i].z * r, hr[i].w * r);
        }
        if (tile + (int)gridDim.x < ntiles) load_tile(tile + gridDim.x);
        __syncthreads();

        {
            const int lane = tile_thread() & 63, li = lane & 15, lq = lane >> 4;
            const int ucol = 16 * ht + 4 * lq;           // first of this lane's four units
            // ---- phase 1: the three gates of this wave's hidden tile
            f4 az[RTW], ar[RTW], ah[RTW];
            float sx[RTW], sh[RTW];
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const int row = 16 * q + li;
                az[q] = ar[q] = ah[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < KCX; ++kc) {
                    const f8x8 a = mma_fp8_operand(&sX[row * LDX + kc * KC + lq * KQ]);
                    az[q] = mma_fp8(az[q], wz[kc], a);
                    ar[q] = mma_fp8(ar[q], wr[kc], a);
                    ah[q] = mma_fp8(ah[q], wh[kc], a);
                }
                const f4 rs = *reinterpret_cast<const f4 *>(&sRow[4 * row]);
                sx[q] = rs.x;
                sh[q] = rs.y;
                az[q] *= rs.z;
                ar[q] *= rs.z;
#pragma unroll
                for (int kh = 0; kh < HC; ++kh) {
                    const f8x8 a = mma_fp8_operand(&sQ[row * LDQ + kh * KC + lq * KQ]);
                    az[q] = mma_fp8(az[q], wz[KCX + kh], a);
                    ar[q] = mma_fp8(ar[q], wr[KCX + kh], a);
                }
            }
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const int row = 16 * q + li;
                const f4 hold = *reinterpret_cast<const f4 *>(&sH[row * LDS32 + ucol]);
                const f4 sz = scales(ucol), sr = scales(H + ucol), sc = scales(2 * H + ucol);
                float m = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    az[q][e] = sigmoid(az[q][e] * sh[q] * sz[e]);
                    ar[q][e] = sigmoid(ar[q][e] * sh[q] * sr[e]) * hold[e];   // r*h
                    ah[q][e] *= sx[q] * sc[e];
                    m = fmaxf(m, fabsf(ar[q][e]));
                }
                wave_max(m, row, lq);
            }
            __syncthreads();
            float srh[RTW];
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const int row = 16 * q + li;
                const float m = row_max(row), r = 448.0f / m;
                srh[q] = m / 448.0f;
                *reinterpret_cast<uint32_t *>(&sQ[row * LDQ + ucol]) =
                    pack4_e4m3(ar[q][0] * r, ar[q][1] * r, ar[q][2] * r, ar[q][3] * r);
            }
            __syncthreads();

            // ---- phase 2: U_h (r*h); new state
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const int row = 16 * q + li;
                f4 au = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < HC; ++kc) au = mma_fp8(au, W2R ? w2[W2R ? kc : 0] : sW2[W2R ? 0 : (ht * HC + kc) * 64 + lane],
                                 mma_fp8_operand(&sQ[row * LDQ + kc * KC + lq * KQ]));
                const f4 su = scales(3 * H + ucol);
                const f4 hold = *reinterpret_cast<const f4 *>(&sH[row * LDS32 + ucol]);
                float m = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float z = az[q][e];
                    const float c = fast_tanh(ah[q][e] + au[e] * srh[q] * su[e]);
                    const float hn = c + z * (hold[e] - c);   // z h + (1 - z) c
                    az[q][e] = hn;
                    m = fmaxf(m, fabsf(hn));
                }
                if (row < nrows) *(__attribute__((address_space(1))) f4 *)(hg + row * H + ucol) = az[q];
                wave_max(m, row, lq);
            }
            __syncthreads();
            float shp[RTW];
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const int row = 16 * q + li;
                const float m = row_max(row), r = 448.0f / m;
                shp[q] = m / 448.0f;
                *reinterpret_cast<uint32_t *>(&sHp[row * LDQ + ucol]) =
                    pack4_e4m3(az[q][0] * r, az[q][1] * r, az[q][2] * r, az[q][3] * r);
            }
            __syncthreads();

            // ---- MLP head
            const uint8_t *src = sHp;
            const f8x8 *Wo = sW3;
            constexpr int CO = HM > 0 ? MC : HC;             // k-chunks of the output layer
            float sin_[RTW];
#pragma unroll
            for (int q = 0; q < RTW; ++q) sin_[q] = shp[q];
            if constexpr (HM > 0) {
                const f4 s3u = scales(4 * H + ucol);
#pragma unroll
                for (int q = 0; q < RTW; ++q) {
                    const int row = 16 * q + li;
                    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kc = 0; kc < HC; ++kc)
                        acc = mma_fp8(acc, sW3[(ht * HC + kc) * 64 + lane], mma_fp8_operand(&sHp[row * LDQ + kc * KC + lq * KQ]));
                    float m = 0.0f;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        ar[q][e] = fmaxf(acc[e] * shp[q] * s3u[e], 0.f);
                        m = fmaxf(m, ar[q][e]);
                    }
                    wave_max(m, row, lq);
                }
                __syncthreads();
#pragma unroll
                for (int q = 0; q < RTW; ++q) {
                    const int row = 16 * q + li;
                    const float m = row_max(row), r = 448.0f / m;
                    sin_[q] = m / 448.0f;
                    *reinterpret_cast<uint32_t *>(&sAm[row * LDQ + ucol]) =
                        pack4_e4m3(ar[q][0] * r, ar[q][1] * r, ar[q][2] * r, ar[q][3] * r);
                }
                __syncthreads();
                src = sAm;
                Wo = sW4;
            }
            for (int ot = ht; ot < OT; ot += HT) {
                const int oc = 16 * ot + 4 * lq;
                const f4 so4 = scales(SO + oc);
#pragma unroll
                for (int q = 0; q < RTW; ++q) {
                    const int row = 16 * q + li;
                    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kc = 0; kc < CO; ++kc)
                        acc = mma_fp8(acc, Wo[(ot * CO + kc) * 64 + lane], mma_fp8_operand(&src[row * LDQ + kc * KC + lq * KQ]));
                    // nout is even: the pairs (oc, oc+1), (oc+2, oc+3) are inside or outside together
                    if (row < nrows) {
                        typedef float v2 __attribute__((ext_vector_type(2)));
                        typedef __attribute__((address_space(1))) v2 gv2;
                        gfloat *o = dp + row * nout + oc;
                        if (oc < nout) *(gv2 *)o = v2{acc[0] * sin_[q] * so4[0], acc[1] * sin_[q] * so4[1]};
                        if (oc + 2 < nout) *(gv2 *)(o + 2) = v2{acc[2] * sin_[q] * so4[2], acc[3] * sin_[q] * so4[3]};
                    }
                }
            }
        }
    }
}

// Persistent BF16 kernel for the shapes k_net_reg does not cover (H = 128, or
// H = 64 at K = 3; standard rows, Hm = 0 or H).  One wave per hidden tile, for
// all rows of a tile, with that hidden tile's gate fragments in registers for
// the whole launch: 164 VGPRs at K = 3, H = 128, where the eight waves hold 336 KB
// of weights and LDS the 110 KB of U_h, of the MLP and of the output beside a
// tile's rows.  The next tile's input rows and FP32 state (in the update's lane
// layout) are requested as soon as their registers are free.
// At K = 3 that leaves LDS for 32 rows; at K <= 2 64 rows fit and are faster
// (835 x 288, K = 2, step 180 us against 188).
// Bound, with 64 flows of 128 x 128 patches at K = 3 and H = 128 (2.4 GB), by the LDS
// reads of the operands: all eight waves read every row fragment, 68 KB per
// wave and tile.  600 us; with fragments streamed from L2 for 128 rows at a
// time 728; with each fragment read just before its products, as the compiler
// orders them, 630; with both row tiles' output fragments read by each wave 610.
// At H = 64 two workgroups of four waves share a CU (512 x 256: step 225 -> 220 us).
// Small grids gain more, as no tile waits for weights: step times at 30 x 20 patches
// and K = 3, H = 128 38.3 -> 27.4 us (30.4 with the streamed kernel), H = 64
// 30.2 -> 24.6.
constexpr int wide_rows(int K) { return K <= 2 ? 64 : 32; }
// Instruction order: N times M matrix products, then one LDS read.
template <int N, int M>
__device__ __forceinline__ void mfma_then_read()
{
    if constexpr (N > 0) {
        __builtin_amdgcn_sched_group_barrier(0x008, M, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        mfma_then_read<N - 1, M>();
    }
}
// Workgroup barrier for LDS data only: this wave's LDS accesses complete,
// then s_barrier; outstanding global loads and stores stay in flight.  (The
// memory clobber keeps the compiler from moving memory accesses across it.)
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int K, int H, int HM>
__global__ __launch_bounds__(4 * H, 2) void k_net_wide(FlowArgs single, const BatchTable *__restrict__ bt,
                                                                  NetArgs net, int ntiles)
{
    typedef Op<1> O;
    constexpr int n = 1 << K, nf = (n + 1) * (n + 1), nin = 4 * nf + 4, nout = 2 * nf;
    constexpr int NT = 4 * H, R = wide_rows(K), RTW = R / 16;
    constexpr int KC = 32, KQ = 8, HT = H / 16, HC = H / KC;
    constexpr int KC1 = (nin + H + KC - 1) / KC, KCX = (nin + KC - 1) / KC;   // k-chunks; those with input columns
    constexpr int OT = (nout + 15) / 16;
    // row pitch: an odd number of 16-byte pieces
    constexpr int LDA = (KC1 * KC / 8) % 2 ? KC1 * KC : KC1 * KC + 8;
    constexpr int LDH = H + 8, PADK = KC1 * KC - nin - H;
    constexpr bool W2R = H == 64;                     // U_h in registers, or in LDS
    constexpr int W2N = W2R ? 1 : HT * HC * 64, W3N = (HM > 0 ? HT : OT) * HC * 64, W4N = HM > 0 ? OT * HC * 64 : 1;
    constexpr int XP = nin / 8, XCH = R * XP, XPT = (XCH + NT - 1) / NT;      // 16-byte pieces of the input rows
    static_assert(HM == 0 || HM == H, "MLP hidden tiles follow the hidden tiles");
    static_assert(nin % 8 == 0 && (H == 64 || H == 128), "rows in 16-byte pieces");
    if (bt) ntiles = bt->prefix[kKindNet][bt->nflows];   // batched: the table's row tiles
    ntiles *= 64 / R;                                    // this kernel's tiles

    __shared__ __align__(16) __bf16 sA[R * LDA];      // [x | h | 0]
    __shared__ __align__(16) __bf16 sG[R * LDH];      // r * h, then the MLP hidden layer
    __shared__ __align__(16) __bf16 sHp[R * LDH];     // h'
    __shared__ __align__(16) bf8 sW2[W2N];
    __shared__ __align__(16) bf8 sW3[W3N];
    __shared__ __align__(16) bf8 sW4[W4N];

    const int tid = threadIdx.x, ht = __builtin_amdgcn_readfirstlane(tid >> 6), lane0 = tid & 63;
    const bf8 *B1 = reinterpret_cast<const bf8 *>(net.B1);
    const bf8 *B2 = reinterpret_cast<const bf8 *>(net.B2);
    const bf8 *B3 = reinterpret_cast<const bf8 *>(net.B3);
    const bf8 *B4 = reinterpret_cast<const bf8 *>(net.B4);
    // (the candidate's weights are zero in the chunks of state alone)
    bf8 wz[KC1], wr[KC1], wh[KCX], w2[W2R ? HC : 1];
#pragma unroll
    for (int kc = 0; kc < KC1; ++kc) {
        wz[kc] = B1[((0 * HT + ht) * KC1 + kc) * 64 + lane0];
        wr[kc] = B1[((1 * HT + ht) * KC1 + kc) * 64 + lane0];
    }
#pragma unroll
    for (int kc = 0; kc < KCX; ++kc) wh[kc] = B1[((2 * HT + ht) * KC1 + kc) * 64 + lane0];
    if constexpr (W2R) {
#pragma unroll
        for (int kc = 0; kc < HC; ++kc) w2[kc] = B2[(ht * HC + kc) * 64 + lane0];
    } else {
        for (int t = tid; t < W2N; t += NT) sW2[t] = B2[t];
    }
    for (int t = tid; t < W3N; t += NT) sW3[t] = B3[t];
    if (HM > 0)
        for (int t = tid; t < W4N; t += NT) sW4[t] = B4[t];
    // the k-padding columns stay zero for the whole launch
    if (PADK > 0)
        for (int t = tid; t < R * PADK; t += NT) sA[(t / PADK) * LDA + nin + H + t % PADK] = (__bf16)0.f;

    // A tile's buffers.  The fields are read in two branches: a pointer that
    // may point at either the kernel argument or the batch table would make
    // them flat loads (and the lambdas below would reach the argument through
    // a generic pointer).
    typedef __attribute__((address_space(1))) float gfloat;
    struct Rows {
        gptr<bf8> X;
        gfloat *h, *dp;
        int nrows;                                       // (none or negative: the second half of a short row tile)
    };
    const void *const s_X = single.X;
    float *const s_h = single.h, *const s_dp = single.dpatch;
    const int s_P = single.nx * single.ny;
    auto rows_of = [&](int tile) -> Rows {
        int blk = tile / (64 / R);
        const void *X;
        float *h, *dp;
        int P;
        if (bt) {
            const FlowArgs &F = *batch_flow(bt, kKindNet, blk);
            X = F.X; h = F.h; dp = F.dpatch; P = F.nx * F.ny;
        } else {
            X = s_X; h = s_h; dp = s_dp; P = s_P;
        }
        const int row0 = blk * 64 + R * (tile % (64 / R));
        Rows r;
        r.X = (gptr<bf8>)(reinterpret_cast<const __bf16 *>(X) + (size_t)row0 * nin);
        r.h = (gfloat *)(h + (size_t)row0 * H);
        r.dp = (gfloat *)(dp + (size_t)row0 * nout);
        r.nrows = min(R, P - row0);
        return r;
    };
    // The next tile's rows: input pieces and, in the lane layout of the update
    // (rows 16 q + li, units ucol .. ucol + 3), the FP32 state.  Rows past the
    // flow's end read its last row.
    bf8 xr[XPT];
    f4 hold[RTW];
    auto load_x = [&](const Rows &rw) {
        const int t0 = tile_thread();
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int c = t0 + i * NT;
            xr[i] = rw.X[tile_piece(c, XP, rw.nrows)];
        }
    };
    auto load_hold = [&](const Rows &rw) {
        const int l = tile_thread() & 63;
#pragma unroll
        for (int q = 0; q < RTW; ++q)
            hold[q] = *(const __attribute__((address_space(1))) f4 *)(rw.h + tile_row(16 * q + (l & 15), rw.nrows) * H +
                                                                       16 * ht + 4 * (l >> 4));
    };
    Rows rw{};
    if ((int)blockIdx.x < ntiles) {
        rw = rows_of(blockIdx.x);
        load_x(rw);
        load_hold(rw);
    }

    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int nrows = rw.nrows;
        gfloat *const hg = rw.h;
        gfloat *const dp = rw.dp;
        // (the last tile repeats its own loads; the rows staged here were last
        // read before the previous tile's second barrier)
        if (tile + (int)gridDim.x < ntiles) rw = rows_of(tile + gridDim.x);
        const int t1 = tile_thread();
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int c = t1 + i * NT;
            if (c < XCH) *reinterpret_cast<bf8 *>(&sA[(c / XP) * LDA + 8 * (c % XP)]) = xr[i];
        }
        const int lane = t1 & 63, li = lane & 15, lq = lane >> 4, ucol = 16 * ht + 4 * lq;
#pragma unroll
        for (int q = 0; q < RTW; ++q) {
            bf4 hb;
            hb[0] = (__bf16)hold[q].x; hb[1] = (__bf16)hold[q].y; hb[2] = (__bf16)hold[q].z; hb[3] = (__bf16)hold[q].w;
            *reinterpret_cast<bf4 *>(&sA[(16 * q + li) * LDA + nin + ucol]) = hb;
        }
        load_x(rw);
        lds_barrier();

        // ---- the three gates of this wave's hidden tile
        f4 az[RTW], ar[RTW], ah[RTW];
#pragma unroll
        for (int q = 0; q < RTW; ++q) az[q] = ar[q] = ah[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < KC1; ++kc)
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const bf8 a = *reinterpret_cast<const bf8 *>(&sA[(16 * q + li) * LDA + kc * KC + lq * KQ]);
                az[q] = O::mma(az[q], wz[kc], a);
                ar[q] = O::mma(ar[q], wr[kc], a);
                if (kc < KCX) ah[q] = O::mma(ah[q], wh[kc], a);
            }
        // (fragments are read four ahead of their products)
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
        mfma_then_read<RTW * KCX, 3>();
        mfma_then_read<RTW * (KC1 - KCX) - 4, 2>();
#pragma unroll
        for (int q = 0; q < RTW; ++q) {
            bf4 rh;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                az[q][e] = sigmoid_l2(az[q][e]);
                rh[e] = (__bf16)(sigmoid_l2(ar[q][e]) * hold[q][e]);
            }
            *reinterpret_cast<bf4 *>(&sG[(16 * q + li) * LDH + ucol]) = rh;
        }
        // (weights from LDS are read before the barrier that their products wait at)
        bf8 wu[HC];
#pragma unroll
        for (int kc = 0; kc < HC; ++kc) wu[kc] = W2R ? w2[W2R ? kc : 0] : sW2[W2R ? 0 : (ht * HC + kc) * 64 + lane];
        lds_barrier();

        // ---- U_h (r * h); new state
#pragma unroll
        for (int q = 0; q < RTW; ++q) {
            const int r = 16 * q + li;
            f4 au = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < HC; ++kc)
                au = O::mma(au, wu[kc], *reinterpret_cast<const bf8 *>(&sG[r * LDH + kc * KC + lq * KQ]));
            f4 hn;
            bf4 hb;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float z = az[q][e];
                // h' = z h + (1 - z) c = c + z (h - c), c the candidate state
                const float c = tanh_l2(ah[q][e] + au[e]);
                hn[e] = c + z * (hold[q][e] - c);
                hb[e] = (__bf16)hn[e];
            }
            if (r < nrows) *(__attribute__((address_space(1))) f4 *)(hg + r * H + ucol) = hn;
            *reinterpret_cast<bf4 *>(&sHp[r * LDH + ucol]) = hb;
        }
        load_hold(rw);
        bf8 wm[HC];
        if constexpr (HM > 0) {
#pragma unroll
            for (int kc = 0; kc < HC; ++kc) wm[kc] = sW3[(ht * HC + kc) * 64 + lane];
        }
        lds_barrier();

        // ---- MLP head
        const __bf16 *src = sHp;
        if constexpr (HM > 0) {
#pragma unroll
            for (int q = 0; q < RTW; ++q) {
                const int r = 16 * q + li;
                f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kc = 0; kc < HC; ++kc)
                    acc = O::mma(acc, wm[kc], *reinterpret_cast<const bf8 *>(&sHp[r * LDH + kc * KC + lq * KQ]));
                bf4 m;
#pragma unroll
                for (int e = 0; e < 4; ++e) m[e] = (__bf16)fmaxf(acc[e], 0.f);
                *reinterpret_cast<bf4 *>(&sG[r * LDH + ucol]) = m;
            }
            lds_barrier();
            src = sG;
        }
        // half of the waves take each row tile, and read its rows once for all
        // their output tiles
        static_assert(HT % RTW == 0, "a row tile for each group of waves");
        const int r = 16 * (ht % RTW) + li;
        bf8 ao[HC];
#pragma unroll
        for (int kc = 0; kc < HC; ++kc) ao[kc] = *reinterpret_cast<const bf8 *>(&src[r * LDH + kc * KC + lq * KQ]);
#pragma unroll
        for (int j = 0; j < (OT + HT / RTW - 1) / (HT / RTW); ++j) {
            const int ot = ht / RTW + j * (HT / RTW), oc = 16 * ot + 4 * lq;
            if (ot >= OT) break;
            f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kc = 0; kc < HC; ++kc)
                acc = O::mma(acc, HM > 0 ? sW4[HM > 0 ? (ot * HC + kc) * 64 + lane : 0] : sW3[(ot * HC + kc) * 64 + lane], ao[kc]);
            // nout is even: the pairs (oc, oc+1), (oc+2, oc+3) are inside or outside together
            if (r < nrows) {
                gfloat *o = dp + r * nout + oc;
                typedef float v2 __attribute__((ext_vector_type(2)));
                typedef __attribute__((address_space(1))) v2 gv2;
                if (oc < nout) *(gv2 *)o = v2{acc[0], acc[1]};
                if (oc + 2 < nout) *(gv2 *)(o + 2) = v2{acc[2], acc[3]};
            }
        }
    }
}

// k_net_wide and k_net_q8p take rows of the standard width 4 nf + 4 and the GRU as
// printed.
static bool standard_rows(const NetArgs &net)
{
    const int n = 1 << net.K;
    return net.nin == 4 * (n + 1) * (n + 1) + 4 && !net.reset_after;
}
// k_net_reg takes the paper's rows and the reset after U_h as well; H = 32 and 96 at
// K = 3, what k_net_wide leaves out at H = 128 or K = 3, and other MLP widths run the
// streamed kernel.
static bool use_reg(const NetArgs &net)
{
    return net.prec == 1 && net.K <= 2 && net.H <= 96 && (net.Hm == 0 || net.Hm == net.H) &&
           (net.nin == 40 || net.nin == 56 || net.nin == 104);
}
static bool use_q8p(const NetArgs &net)
{
    return standard_rows(net) && net.prec == 2 && (net.H == 64 || net.H == 128) && (net.Hm == 0 || net.Hm == net.H);
}
int num_cus()
{
    // (a constant of the machine, read once)
    static const int cus = [] {
        int dev = 0, n = 0;
        (void)hipGetDevice(&dev);
        return hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess ? n : 256;
    }();
    return cus;
}
static bool use_wide(const NetArgs &net)
{
    return standard_rows(net) && net.prec == 1 && !use_reg(net) && (net.H == 64 || net.H == 128) &&
           (net.Hm == 0 || net.Hm == net.H);
}

template <int PREC, int H, int R, bool BATCHED>
static hipError_t launch_net_r(const FlowArgs &f, const BatchTable *bt, int nblocks, const NetArgs &net, hipStream_t s)
{
    const int lds = stream_rows<PREC, H, R>(net.kc1, net.Hm).bytes;
    hipLaunchKernelGGL((k_net<PREC, H, R, BATCHED>), dim3(nblocks), dim3(64 * stream_waves<H, R>()), lds, s, f, bt, net);
    return hipGetLastError();
}

template <int PREC, int H>
static hipError_t launch_net_t(const FlowArgs &f, const BatchTable *bt, int ntiles, const NetArgs &net,
                               hipStream_t s)
{
    if (bt) return launch_net_r<PREC, H, 64, true>(f, bt, ntiles, net, s);
    // few patches: 16 a workgroup, up to two workgroups per CU.  Step times (us, 64
    // against 16) in FP32: K = 2, H = 64 2400 patches 33.1 / 25.4, 8192 35.2 / 30.8, 16384
    // 37.4 / 39.7; K = 1, H = 32 256 patches 23.4 / 22.0, 8192 25.1 / 24.9; K = 3, H = 128
    // 60 patches 76.3 / 39.8, 8192 86.4 / 67.0, 16384 97.8 / 113.0.  BF16 with an MLP of 256:
    // 600 patches 24.4 / 22.3, 8192 26.4 / 25.3, 20000 33.2 / 36.1.
    const int P = f.nx * f.ny;
    if (P <= 2 * kFewRows * num_cus()) return launch_net_r<PREC, H, kFewRows, false>(f, bt, (P + kFewRows - 1) / kFewRows, net, s);
    return launch_net_r<PREC, H, 64, false>(f, bt, ntiles, net, s);
}

hipError_t launch_net(const FlowArgs &f, const BatchTable *bt, int ntiles, const NetArgs &net, hipStream_t s)
{
    // persistent kernels: a grid that fills the CUs, or one tile per workgroup
    auto grid = [&](int tiles, int per_cu) { return dim3(tiles < per_cu * num_cus() ? tiles : per_cu * num_cus()); };
    // With at most 16 patches per CU a workgroup of the persistent kernels has
    // one tile for the weights it loads; from H = 96 on the streamed kernel's
    // 16-patch tiles are then faster (step us, persistent against streamed): K = 2,
    // H = 96 400 patches 23.9 / 22.3, 2400 24.7 / 22.5, 6000 25.5 / 25.3, 12288 27.6 / 30.6;
    // K = 2, H = 128 2400 26.0 / 23.0; K = 3, H = 128 2400 27.7 / 26.6, 6000 33.7 / 35.0.  At H = 32
    // and 64 they are level (K = 2, H = 64 400 patches 22.3 / 22.5, 2400 22.9 / 22.0; K = 3,
    // H = 64 24.7 / 25.2).
    const bool few = !bt && net.H >= 96 && f.nx * f.ny <= kFewRows * num_cus();
    if (!few && use_reg(net)) {
        // (at H = 32 a workgroup is four waves of up to 210 registers: two per CU)
        const dim3 g = grid(ntiles, net.H == 32 ? 2 : 1);
#define DNNMG_REG(NN, HH)                                                                                              \
        if (net.nin == NN && net.H == HH) {                                                                            \
            hipLaunchKernelGGL((k_net_reg<NN, HH>), g, dim3(net_reg_threads<HH>()), 0, s, f, bt, net, ntiles); \
            return hipGetLastError();                                                                                  \
        }
        DNNMG_REG(40, 32) DNNMG_REG(56, 32) DNNMG_REG(104, 32)
        DNNMG_REG(40, 64) DNNMG_REG(56, 64) DNNMG_REG(104, 64)
        DNNMG_REG(40, 96) DNNMG_REG(56, 96) DNNMG_REG(104, 96)
#undef DNNMG_REG
        return hipErrorInvalidValue;
    }
    if (!few && use_wide(net)) {
        const dim3 g = grid(ntiles * (64 / wide_rows(net.K)), 128 / net.H), b(4 * net.H);
#define DNNMG_WIDE(KK, HH, MM)                                                                             \
        if (net.K == KK && net.H == HH && net.Hm == MM) {                                                 \
            hipLaunchKernelGGL((k_net_wide<KK, HH, MM>), g, b, 0, s, f, bt, net, ntiles);                 \
            return hipGetLastError();                                                                     \
        }
        DNNMG_WIDE(1, 128, 0) DNNMG_WIDE(1, 128, 128)
        DNNMG_WIDE(2, 128, 0) DNNMG_WIDE(2, 128, 128)
        DNNMG_WIDE(3, 64, 0) DNNMG_WIDE(3, 64, 64)
        DNNMG_WIDE(3, 128, 0) DNNMG_WIDE(3, 128, 128)
#undef DNNMG_WIDE
        return hipErrorInvalidValue;
    }
    if (use_q8p(net)) {
        // as many workgroups of H / 16 waves as a CU's four SIMDs hold
        const dim3 g = grid(ntiles * (64 / kQ8Rows), 64 * q8p_waves(net.K) / net.H), b(4 * net.H);
#define DNNMG_Q8P(KK, HH, MM) hipLaunchKernelGGL((k_net_q8p<KK, HH, MM>), g, b, 0, s, f, bt, net, ntiles)
#define DNNMG_Q8P_H(KK)                                                                            \
        if (net.H == 64) { if (net.Hm == 64) DNNMG_Q8P(KK, 64, 64); else DNNMG_Q8P(KK, 64, 0); }    \
        else { if (net.Hm == 128) DNNMG_Q8P(KK, 128, 128); else DNNMG_Q8P(KK, 128, 0); }
        switch (net.K) {
        case 1: DNNMG_Q8P_H(1) break;
        case 2: DNNMG_Q8P_H(2) break;
        case 3: DNNMG_Q8P_H(3) break;
        default: return hipErrorInvalidValue;
        }
#undef DNNMG_Q8P_H
#undef DNNMG_Q8P
        return hipGetLastError();
    }
    if (net.prec == 2) {
        dim3 g(ntiles), b(kThreads);
#define DNNMG_FP8_CASE(HH)                                                                  \
        if (net.H == HH) {                                                                  \
            if (bt) hipLaunchKernelGGL((k_net_fp8<HH, true>), g, b, 0, s, f, bt, net);      \
            else hipLaunchKernelGGL((k_net_fp8<HH, false>), g, b, 0, s, f, bt, net);        \
            return hipGetLastError();                                                       \
        }
        DNNMG_FP8_CASE(32)
        DNNMG_FP8_CASE(64)
        DNNMG_FP8_CASE(128)
#undef DNNMG_FP8_CASE
        return hipErrorInvalidValue;
    }
    if (net.prec == 0) {
        if (net.H == 32) return launch_net_t<0, 32>(f, bt, ntiles, net, s);
        if (net.H == 64) return launch_net_t<0, 64>(f, bt, ntiles, net, s);
        if (net.H == 96) return launch_net_t<0, 96>(f, bt, ntiles, net, s);
        if (net.H == 128) return launch_net_t<0, 128>(f, bt, ntiles, net, s);
    } else if (net.prec == 1) {
        if (net.H == 32) return launch_net_t<1, 32>(f, bt, ntiles, net, s);
        if (net.H == 64) return launch_net_t<1, 64>(f, bt, ntiles, net, s);
        if (net.H == 96) return launch_net_t<1, 96>(f, bt, ntiles, net, s);
        if (net.H == 128) return launch_net_t<1, 128>(f, bt, ntiles, net, s);
    }
    return hipErrorInvalidValue;
}


}  // namespace dnnmg
