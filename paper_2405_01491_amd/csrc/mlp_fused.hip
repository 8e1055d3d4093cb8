// Fused species network: forward, head and adjoint of the
// 1008-256-192-160-1 CELU network (Sec. 2.2, "Neural Networks"; Sec. 2.4)
// for one tile of TM same-species atoms in a single kernel.
//
//   h1 = CELU(W1 a + b1), h2 = CELU(W2 h1 + b2), h3 = CELU(W3 h2 + b3)
//   E  = w4 . h3 + b4
//   d3 = w4 * CELU'(h3), d2 = (W3^T d3) * CELU'(h2), d1 = (W2^T d2) * CELU'(h1)
//   dE/da = W1^T d1
//
// Four waves split every layer's output columns (64 / 48 / 48 per wave; the
// 160-wide layer is padded to 192 with zero weights).  Every product is
// computed transposed, weights as the first MFMA operand and atoms as the
// second, so that a lane ends up with four consecutive columns of one atom:
// the epilogues store activations 8 bytes, gradients 16 bytes at a time, and
// everything per atom (scales, head sum) is one value per lane.  Each wave
// keeps its h1 and h2 columns in registers (MFMA accumulator layout) for the
// CELU' epilogues of the adjoint, which produces exactly the same columns.
// The activations of every layer pass through one LDS tile; the first layer
// streams the AEV tile through a double-buffered part of the same LDS.
// Weights are pre-packed per species in MFMA fragment order, so a lane
// fetches its fragment with 16-byte loads; each wave reads only its own
// columns.  Only the AEV tile is read from and dE/dAEV written to HBM.
//
//   BF16 form: v_mfma_f32_16x16x32_bf16, inputs rounded to bfloat16, float32
//     accumulation.
//   FP32 form: v_mfma_f32_16x16x32_f16 on inputs split into float16 numbers,
//     x s = hi + lo with s a power of two (hi the nearest float16 of x s, lo
//     that of the remainder); weights also keep what hi + lo leaves, so that
//     all of their 24 bits count.  Four products per step, rest*hi + lo*hi +
//     hi*lo + hi*hi, into float32 accumulators.  s is taken per product from
//     the largest magnitude: for an atom's input row, measured each time, and
//     for a species' weight matrix, once when it is packed; the largest element
//     then lies in [2^14, 2^15).  Weights down to 2^-15 of it are whole, and
//     smaller ones off by at most 2^-39 of it; inputs down to 2^-17 of the
//     largest keep 22 to 24 bits, smaller ones are off by at most 2^-39 of it.
//     One step replaces eight v_mfma_f32_16x16x4_f32 (256 cycles) by four
//     products of 16 cycles, and rounds a sum four times where that rounded 32
//     times.  Error (rms) against 64 bits over six sets of weights (uniform,
//     normal, heavy-tailed, biased), water and organic boxes, beside the float32
//     MFMAs': atomic energies 3.0e-8 of their terms (4.3e-8), the mean of a
//     species' energies 4.4e-9 (4.3e-9; largest 1.0e-8, 1.3e-8), a box's energy
//     3.0e-9 (3.2e-9), dE/dAEV 3.0e-7 (4.7e-7), its sum over a box 0.7e-7
//     (1.3e-7); over ten sets, a box's virial 3.3e-8 of its atoms' (6.3e-8).
//     The fourth product takes a fifth to a quarter more time: 184 and 220 us
//     at 99,999 water atoms, 57 and 71 us at 6,001 dense ones (float32 MFMAs:
//     440, 122).
//
// A non-finite input makes its atom's results NaN, and no other atom's.
#include <cmath>
#include <cstring>
#include <type_traits>

#include "nnp_internal.hpp"

namespace nnp {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// Read through a global-address-space pointer: a generic (flat) load would
// also count against the LDS wait counter.
typedef __attribute__((address_space(1))) const f32x4 gfloat4;

constexpr int K0 = 1024, N1 = 256, N2 = 192, N3 = 192;
constexpr int NW = 4, kThreads = NW * kWave;   // waves of a tile
constexpr int NC1 = N1 / 16 / NW, NC2 = N2 / 16 / NW;   // a wave's column blocks: w + NW i
static_assert(N3 == N2, "layers two and three share their column split");
constexpr int KS = 32;                 // k per step (one MFMA's)
constexpr int LD = N1 + 8;             // row stride of an LDS plane (elements)
// first layer: k-steps per chunk
template <bool BF>
constexpr int chunk_steps() { return BF ? 8 : 4; }
constexpr int kRad = 7;                // radial feature blocks of 16 (one per species)

// The weight packs of one species, one after the other: forward of the layers
// one to three, adjoint of three to one, each K x N.
enum { kF1, kF2, kF3, kA3, kA2, kA1, kPacks };
constexpr int kPackK[kPacks] = {K0, N1, N2, N3, N2, N1};
constexpr int kPackN[kPacks] = {N1, N2, N3, N2, N1, K0};
constexpr int pack_first(int q) {   // fragments of 512 weights
    return q == 0 ? 0 : pack_first(q - 1) + kPackK[q - 1] * kPackN[q - 1] / 512;
}

// planes of an operand: hi and lo float16 (FP32 form), or one bfloat16
template <bool BF>
constexpr int planes() { return BF ? 1 : 2; }
// bytes of a packed fragment: two float16 and four bits a weight (FP32 form), or
// one bfloat16
template <bool BF>
constexpr int frag_bytes() { return BF ? 1024 : 2048 + 256; }

// CELU and its derivative, without branches.  FP32 form: with e = exp(min(v, 0)
// / alpha), which is exactly 1 for v >= 0, CELU(v) = max(v, 0) + alpha (e - 1),
// of which one term is zero, and CELU'(v) = e.  BF16 form: the derivative from
// the output, h > 0 ? 1 : 1 + h / alpha (its results are rounded to bfloat16,
// so that the last bit of h decides some of them: the expressions stay as they
// are).  A NaN stays one (fminf would make it 0).  CeluConst: alpha, 1 / alpha,
// and log2(e) / alpha as the sum of two positive floats (one float's error, the
// same for every atom, would bias their sum; v = -inf gives e = 0).
struct CeluConst {
    float a, ia, k_hi, k_lo;
};
struct Celu {
    float h, d;
};
template <bool BF>
__device__ __forceinline__ Celu celu(float v, const CeluConst& c) {
    const float x = v > 0.f ? 0.f : v;
    if constexpr (BF) {
        const float neg = c.a * (__expf(x * c.ia) - 1.f);
        const float h = v > 0.f ? v : neg;
        return {h, h > 0.f ? 1.f : fmaf(h, c.ia, 1.f)};
    } else {
        const float e = __builtin_amdgcn_exp2f(fmaf(x, c.k_hi, x * c.k_lo));
        return {fmaxf(v, 0.f) + fmaf(c.a, e, -c.a), e};
    }
}

// The power of two that takes a largest magnitude m to [2^14, 2^15) (below
// 2^-112 and at zero: 2^126), and its inverse.
struct Pow2 {
    float s, inv;
};
__host__ __device__ __forceinline__ Pow2 pow2_scale(float m) {
    const unsigned e = __builtin_bit_cast(unsigned, m) >> 23;   // m >= 0
    const unsigned b = e > 15u ? 268u - e : 253u;
    return {__builtin_bit_cast(float, b << 23), __builtin_bit_cast(float, (254u - b) << 23)};
}

// The float16 MFMA drops the bits below its widest term's by rounding down, so
// that a sum comes out low by about 1.5e-8 of the sum of its terms' magnitudes,
// whatever its sign.  The packs of the FP32 form therefore hold half of the
// columns negated, and this sign goes into their scale, so that these columns
// err upwards: those with an odd number of ones among the four low bits of
// their index, a sequence that leaves no mean and no trend over the shells of a
// feature block.  (Over ten sets of weights, the networks' part of a box's
// virial: 3.3e-8 of its atoms'; without the signs 1.1e-7; float32 MFMAs 6.3e-8.)
template <bool BF>
__host__ __device__ __forceinline__ float col_sign(int n) { return !BF && (0x6996 >> (n & 15) & 1) ? -1.f : 1.f; }

// One operand fragment: 16 rows (or columns) x 32 k, per plane 8 values per
// lane; of weights with the remainders (FP32 form)
template <bool BF>
struct Frag {
    u16x8 p[planes<BF>()];
};
template <bool BF>
struct WFrag : Frag<BF> {};
template <>
struct WFrag<false> : Frag<false> {
    unsigned r;
};

// Activation fragments of k-step ks (LDS planes `plane` elements apart, row stride ld)
template <bool BF, int MB>
__device__ __forceinline__ void load_a(const uint16_t* act, int plane, int ld, int ks, Frag<BF> (&a)[MB]) {
    const int l = lane_id();
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int p = 0; p < planes<BF>(); ++p)
            a[mb].p[p] = *(const u16x8*)(act + p * plane + (16 * mb + (l & 15)) * ld + KS * ks + 8 * (l >> 4));
}

// The MFMAs of one k-step, smallest products first: acc[mb][nb] += (W[step, nb])^T A[16 mb.., step]^T, or (kAtoms) the
// transpose A W, atoms along the accumulator's rows.
template <bool BF>
__device__ __forceinline__ f32x4 mfma(u16x8 b, u16x8 a, f32x4 c) {
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b), __builtin_bit_cast(bf16x8, a), c,
                                                       0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, b), __builtin_bit_cast(f16x8, a), c, 0,
                                                      0, 0);
}

// The remainders of eight weights, from four bits each: of the remainder times
// kRest, a power of two, a float16's exponent field f (2^(f - 15); 0: none).
// Element e's lies at rest_bit(e) (past bit 31 it goes on at bit 0), where a
// rotation brings each pair's fields into place; the odd ones are negative,
// which the scaling back adds.  Eleven operations a fragment; with shifts, and
// the odd signs set apart, sixteen (99,999 water atoms: 228 us, now 220).
constexpr float kRest = 512.f;
constexpr int rest_bit(int e) { return 10 + 16 * (e & 1) + 4 * (e / 2); }
__device__ __forceinline__ u16x8 remainders(unsigned w) {
    constexpr unsigned field = 0x3c003c00u;
    const u32x4 r = {w & field, __builtin_amdgcn_alignbit(w, w, 4) & field, __builtin_amdgcn_alignbit(w, w, 8) & field,
                     __builtin_amdgcn_alignbit(w, w, 12) & field};
    constexpr _Float16 c = (_Float16)(1.f / kRest);
    constexpr f16x8 back = {c, -c, c, -c, c, -c, c, -c};
    return __builtin_bit_cast(u16x8, __builtin_bit_cast(f16x8, r) * back);
}

template <bool BF, int MB, int NCB, bool kAtoms = false>
__device__ __forceinline__ void mfma_kstep(const Frag<BF> (&a)[MB], const WFrag<BF> (&b)[NCB], f32x4 (&acc)[MB][NCB]) {
    constexpr int kProd = BF ? 1 : 3;
    if constexpr (!BF) {
#pragma unroll
        for (int nb = 0; nb < NCB; ++nb) {
            const u16x8 r = remainders(b[nb].r);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                acc[mb][nb] = kAtoms ? mfma<BF>(a[mb].p[0], r, acc[mb][nb]) : mfma<BF>(r, a[mb].p[0], acc[mb][nb]);
        }
    }
    constexpr int pb[3] = {BF ? 0 : 1, 0, 0}, pa[3] = {0, BF ? 0 : 1, 0};
#pragma unroll
    for (int q = 0; q < kProd; ++q)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NCB; ++nb)
                acc[mb][nb] = kAtoms ? mfma<BF>(a[mb].p[pa[q]], b[nb].p[pb[q]], acc[mb][nb])
                                     : mfma<BF>(b[nb].p[pb[q]], a[mb].p[pa[q]], acc[mb][nb]);
}

// A species' packs as a buffer: a load takes a scalar offset beside the lane's,
// so that no address is computed per lane, and is bounds-checked.
typedef __amdgpu_buffer_rsrc_t PackBuf;
template <bool BF>
__device__ __forceinline__ PackBuf pack_buf(const void* packs) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)packs, 0, pack_first(kPacks) * frag_bytes<BF>(), 0x00027000);
}

// Weight fragments of the column blocks blk and k-step ks of pack q:
// [block][k-step][plane][64 lanes][8] (and the remainders' bits)
template <bool BF, int Q, int NCB>
__device__ __forceinline__ void load_b(PackBuf B, const int (&blk)[NCB], int ks, WFrag<BF> (&b)[NCB]) {
    constexpr int NK = kPackK[Q] / KS;
    const int lane = 16 * lane_id();
#pragma unroll
    for (int nb = 0; nb < NCB; ++nb) {
        const int at = (pack_first(Q) + blk[nb] * NK + ks) * frag_bytes<BF>();
#pragma unroll
        for (int p = 0; p < planes<BF>(); ++p)
            b[nb].p[p] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(B, lane + 1024 * p, at, 0));
        if constexpr (!BF)
            b[nb].r = __builtin_amdgcn_raw_buffer_load_b32(B, lane / 4 + 2048, at, 0);
    }
}

// Ring of weight-fragment registers: k-step t lives in slot t % RS and is
// loaded PD k-steps ahead.  The k loops are unrolled and their loads
// unconditional: slots are indexed at compile time, and the waits count
// exactly the loads in flight (a load under a condition would make the next
// wait one for every load, the prefetched ones included).
template <bool BF>
constexpr int ring_ahead() { return BF ? 2 : 1; }
// slots of an unrolled loop; where turns repeat (first layer), a power of two
template <bool BF>
constexpr int ring_slots() { return ring_ahead<BF>() + 1; }
template <bool BF>
constexpr int ring_turn() { return ring_ahead<BF>() == 1 ? 2 : 4; }

// The weight-fragment ring of one product over K rows; start() issues the
// loads of the first k-steps, so that a caller can put them ahead of the
// epilogue and barrier that precede the product (the barrier waits only for
// LDS operations, not for these loads).
// blk: the NCB output column blocks (a negative entry reads block 0; its
// columns are discarded by the caller)
template <bool BF, int Q, int NCB>
struct BPipe {
    static constexpr int NK = kPackK[Q] / KS;
    static constexpr int PD = ring_ahead<BF>(), RS = ring_slots<BF>();
    static_assert(NK >= PD, "");
    WFrag<BF> rb[RS][NCB];
    int blk[NCB];
    // wave w's blocks w + NW i, or those of list
    __device__ __forceinline__ void start(PackBuf B, int w) {
#pragma unroll
        for (int nb = 0; nb < NCB; ++nb) blk[nb] = w + NW * nb;
        first(B);
    }
    __device__ __forceinline__ void start(PackBuf B, const int* list) {
#pragma unroll
        for (int nb = 0; nb < NCB; ++nb) blk[nb] = max(__builtin_amdgcn_readfirstlane(list[nb]), 0);
        first(B);
    }
    __device__ __forceinline__ void first(PackBuf B) {
#pragma unroll
        for (int t = 0; t < PD; ++t) load_b<BF, Q, NCB>(B, blk, t, rb[t]);
    }
};

// The product of a started ring over the K rows: acc (+)= A W.
template <bool BF, int MB, int Q, int NCB, bool kZero = true>
__device__ __forceinline__ void gemm_run(const uint16_t* act, int plane, PackBuf B, BPipe<BF, Q, NCB>& p,
                                         f32x4 (&acc)[MB][NCB]) {
    constexpr int NK = BPipe<BF, Q, NCB>::NK, RS = BPipe<BF, Q, NCB>::RS, PD = BPipe<BF, Q, NCB>::PD;
    if (kZero) {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NCB; ++nb) acc[mb][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        if (ks + PD < NK) load_b<BF, Q, NCB>(B, p.blk, ks + PD, p.rb[(ks + PD) % RS]);
        __builtin_amdgcn_sched_barrier(0);   // keep the prefetches ahead of this step's MFMAs
        Frag<BF> a[MB];
        load_a<BF, MB>(act, plane, LD, ks, a);
        mfma_kstep<BF, MB, NCB, Q == kA1>(a, p.rb[ks % RS], acc);
    }
}

// Four consecutive columns of one row into the LDS planes, times s (FP32 form)
template <bool BF>
__device__ __forceinline__ void put4(uint16_t* dst, int plane, f32x4 v, float s) {
    if constexpr (BF) {
        *(bf16x4*)dst = __builtin_convertvector(v, bf16x4);
    } else {
        const f32x4 y = v * s;
        const f16x4 hi = __builtin_convertvector(y, f16x4);
        *(f16x4*)dst = hi;
        f32x4 lo;   // exact: hi holds the leading bits of v s
#pragma unroll
        for (int k = 0; k < 4; ++k) lo[k] = fmaf(v[k], s, -(float)hi[k]);
        *(f16x4*)(dst + plane) = __builtin_convertvector(lo, f16x4);
    }
}

__device__ __forceinline__ float max4(float m, f32x4 v) {
    return fmaxf(fmaxf(m, fmaxf(fabsf(v[0]), fabsf(v[1]))), fmaxf(fabsf(v[2]), fabsf(v[3])));
}

}  // namespace

// One network's weights for every species (device table, one entry per network).
static_assert(kPacks == kFusedPacks, "");
struct FusedNet {
    struct Species {
        const void* packs;
        const float* vec;     // b1 [N1], b2 [N2], b3 [N3], head weights [N3], zero padded
        float inv[kPacks];    // 1 / each pack's scale (FP32 form)
        float b4;
    } sp[kMaxSpecies];
};

namespace {

struct FusedArgs {
    const FusedNet* nets;            // [n_nets] (device)
    const int32_t* meta;
    const int32_t* row_atom;
    const void* aev;                 // [rows][K0] float32 or bf16
    float* g_out;                    // [rows][K0] float32 or null
    float* E_row;                    // [rows]
    float* E_atomo;                  // [n] atom order or null
    CeluConst celu;
    // ensemble front (kEns): per network, d1 = dE/dh1 as the next product's
    // operand [n_nets][rows][planes][N1], 1 / its row scales [n_nets][rows]
    // (FP32 form), and E [n_nets][rows]
    uint16_t* d1_out;
    float* d1_inv;
    float* E_net;
    int rows;
    // per row, the species present in its atom's environment (bits 0-7
    // radial, 8-15 angular); null: every feature block may be non-zero
    const uint32_t* amask;
};

constexpr int kXcds = 8;   // accelerator complex dies of one MI355X, each with its own L2

// The tile of this block.  A launch's blocks are dealt to the XCDs in turn
// (block b runs on XCD b mod 8); each XCD takes a contiguous range of tiles,
// so that tiles of one species, which stream the same weight packs, share
// an XCD's L2 instead of every L2 holding every species' packs.  The grid
// (x) is padded to a multiple of 8 blocks; the map is a bijection of the
// padded range, and a block past the last tile exits.
__device__ __forceinline__ int xcd_tile(int n_tiles) {
    const int per = (n_tiles + kXcds - 1) / kXcds;
    return (int)(blockIdx.x % kXcds) * per + (int)(blockIdx.x / kXcds);
}

// The species of the tile at row0, and the row past its last atom.  meta: the
// counts [8] and the first rows [8 + ns .. ] of the species' segments, each
// padded to whole tiles (kRad species: the fused shape has no other).
__device__ __forceinline__ int tile_species_of(const int32_t* __restrict__ meta, int row0) {
    int s = 0;
#pragma unroll
    for (int q = 1; q < kRad; ++q)
        if (meta[8 + q] <= row0) s = q;
    return s;
}
__device__ __forceinline__ int segment_end(const int32_t* __restrict__ meta, int s) { return meta[8 + s] + meta[s]; }

// The species present around some atom of the tile rows row0 .. row0 + TM - 1
// below row_end (AEV kernel's masks; uniform over the wave).  Wave-level.
template <int TM>
__device__ __forceinline__ unsigned tile_species(const uint32_t* amask, int row0, int row_end) {
    unsigned m = 0;
    for (int r = lane_id(); r < TM; r += kWave)
        if (row0 + r < row_end) m |= amask[row0 + r];
    unsigned any = 0;
#pragma unroll
    for (int b = 0; b < 16; ++b)
        if (ballot((m >> b) & 1u)) any |= 1u << b;
    return any;
}

// The 16-feature blocks (bit b: features 16 b .. 16 b + 15) that are non-zero
// for an atom with these species around it: a species' radial block when the
// species occurs within Rc_R, the two blocks of a species pair's angular bin
// when both occur within Rc_A.  One lane per block.
__device__ __forceinline__ unsigned long long species_blocks(unsigned m) {
    const int l = lane_id();
    // angular blocks: pair p = (q, u), q <= u, in the order of the rows of an
    // upper triangle of side kRad
    const int p = (l - kRad) >> 1;
    int q = 0, first = 0;
#pragma unroll
    for (int k = 0, o = 0; k < kRad; ++k, o += kRad + 1 - k)
        if (p >= o) {
            q = k;
            first = o;
        }
    const int u = q + p - first;
    const bool on = l < kRad ? (m >> l) & 1u : (l < kRad * (kRad + 2)) && ((m >> (8 + q)) & (m >> (8 + u)) & 1u);
    return ballot(on);
}

// The set blocks of bm in ascending order into list[0 .. n), then -1 up to
// the next multiple of gran (<= 64); returns that padded count.  Wave-level.
__device__ __forceinline__ int block_list(unsigned long long bm, int* list, int gran) {
    const int l = lane_id();
    const bool on = (bm >> l) & 1ull;
    const unsigned long long b = ballot(on);
    const int n = __popcll(b), n_pad = (n + gran - 1) / gran * gran;
    if (on) list[rank_below(b)] = l;
    if (l >= n && l < n_pad) list[l] = -1;
    return n_pad;
}

// Element r of a and b: swaps the odd 16-lane groups of a with the even ones of
// b (their neighbours below); and the upper half of a with the lower half of b.
__device__ __forceinline__ void swap16(f32x4& a, f32x4& b, int r) {
    const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[r]), __float_as_uint(b[r]), false, false);
    a[r] = __uint_as_float(v[0]);
    b[r] = __uint_as_float(v[1]);
}
__device__ __forceinline__ void swap32(f32x4& a, f32x4& b, int r) {
    const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[r]), __float_as_uint(b[r]), false, false);
    a[r] = __uint_as_float(v[0]);
    b[r] = __uint_as_float(v[1]);
}

// dE/dAEV of the tile for its output blocks b (16 columns each; a negative
// block is padding and is not stored), row i times sc[i] into row row_of(i) of
// g (negative: not stored).  acc: atoms along the accumulator's rows, as the
// first layer's adjoint leaves them.  The column blocks are exchanged between
// the 16-lane groups first, so that one store writes 256 bytes of a row (128
// with two blocks) where it wrote 64 bytes of four: 16 rows of 64 bytes a
// store, the transposed products' layout, cost the dense BF16 networks at
// 23,000 atoms 88 us, four 83 us.
template <bool BF, int MB, int NCB, typename F>
__device__ __forceinline__ void store_g(float* g, F row_of, f32x4 (&acc)[MB][NCB], const int* b, const float* sc) {
    static_assert(NCB == 1 || NCB == 2 || NCB == 4, "");
    const int l = lane_id(), grp = l >> 4;
    const int blk = b[grp & (NCB - 1)];
    const float sign = col_sign<BF>(l);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (NCB >= 2) swap16(acc[mb][0], acc[mb][1 % NCB], r);
            if (NCB == 4) {
                swap16(acc[mb][2 % NCB], acc[mb][3 % NCB], r);
                swap32(acc[mb][0], acc[mb][2 % NCB], r);
                swap32(acc[mb][1 % NCB], acc[mb][3 % NCB], r);
            }
#pragma unroll
            for (int nb = 0; nb < NCB; ++nb) {
                // NCB 4: group nb's row; 2: group nb + (lane's half); 1: the lane's group
                const int i = 16 * mb + 4 * (NCB == 4 ? nb : NCB == 2 ? nb + (grp & 2) : grp) + r;
                const int row = row_of(i);
                if (blk >= 0 && row >= 0) g[(size_t)row * K0 + 16 * blk + (l & 15)] = acc[mb][nb][r] * (sc[i] * sign);
            }
        }
}

// The k-steps of the first layer.  FP32 form: the radial blocks are an odd
// number, so step 3 pairs the last of them with a block of zeros, and every
// species pair's two angular blocks share a step (water needs 5 steps, not 8).
// BF16 form: the features in turn (another order of a sum moves its results by
// roundings of what follows).
// Bit t: some block of step t is in bm (bit b: feature block b).
template <bool BF>
__device__ __forceinline__ unsigned step_mask(unsigned long long bm) {
    const unsigned long long rad = (1ull << kRad) - 1;
    const unsigned long long x = BF ? bm : (bm & rad) | ((bm & ~rad) << 1);
    return (unsigned)ballot((x >> (2 * (lane_id() & 31))) & 3ull);
}
// The feature of position i (0 .. 31) of step t; -1: the zero block
template <bool BF>
__host__ __device__ __forceinline__ int step_feature(int t, int i) {
    const int f = KS * t + i;
    return BF || f < 16 * kRad ? f : (f < 16 * (kRad + 1) ? -1 : f - 16);
}

// kDir: features and dE/dAEV are the caller's, float32 rows in atom order, in
// place of the grouped rows of the workspace (no copy into and out of groups).
// kEns: network blockIdx.y of an ensemble; stops after d1 (the adjoint of the
// first layer sums over networks, k_ens_adj1) and writes this network's
// energies to E_net.
template <bool BF, int TM, bool kEns, bool kDir>
__global__ __launch_bounds__(kThreads, TM > 32 ? 2 : 3) void k_mlp_fused(const FusedArgs A) {
    constexpr int NP = planes<BF>();
    constexpr int CS = chunk_steps<BF>(), CLD = CS * KS + 8;   // first layer: a chunk's k-steps and row stride
    constexpr int MB = TM / 16;
    constexpr int kPlane = TM * LD, kCPlane = TM * CLD;
    constexpr int kElems = NP * (kPlane > 2 * kCPlane ? kPlane : 2 * kCPlane);
    __shared__ __attribute__((aligned(16))) uint16_t smem[kElems];
    __shared__ __attribute__((aligned(16))) float epart[TM][NW];
    __shared__ __attribute__((aligned(16))) float rmax[TM][NW];   // per row and wave, the largest magnitude
    uint16_t* const act = smem;
    const int tile = xcd_tile((A.rows + TM - 1) / TM);
    const int row0 = tile * TM;
    if (row0 >= A.rows) return;
    const int s = tile_species_of(A.meta, row0), row_end = segment_end(A.meta, s);
    if (row0 >= row_end) return;   // past the last segment, or segment padding only
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / kWave), l = lane_id();
    const int lr = l & 15, lc = 4 * (l >> 4);    // this lane's row and first column within a 16 x 16 block
    const float lane_sign = col_sign<BF>(lc);    // columns lc + r: this times col_sign(r), r < 4
    const int net = kEns ? blockIdx.y : 0;
    // this network's and species' pointers, loaded once (the table is read-only)
    const FusedNet::Species* __restrict__ sp = &A.nets[net].sp[s];
    const PackBuf wb = pack_buf<BF>(sp->packs);
    const float iw1 = sp->inv[kF1], iw2 = sp->inv[kF2], iw3 = sp->inv[kF3];
    const float ia3 = sp->inv[kA3], ia2 = sp->inv[kA2], ia1 = sp->inv[kA1];
    const float hb4 = sp->b4;

    // ---------------- active feature blocks of the tile
    // A 16-feature block of the AEV (a species' radial shells, or half of a
    // species pair's angular bin) is zero for an atom whose environment lacks
    // that species.  The first layer runs only over the k-steps that hold a
    // block some atom of the tile can have non-zero, and its adjoint only
    // over those output blocks: the skipped products are exact zeros, and
    // dE/dAEV is consumed only where the features are non-zero.  Without a
    // mask every block is active.  A k-step holds the same 32 features in
    // every tile, so that an atom's result does not depend on its tile.
    // Every wave works the mask out for itself, on the scalar unit: the
    // first loads of features and weights wait for no barrier.
    const unsigned long long bm = A.amask ? species_blocks(tile_species<TM>(A.amask, row0, row_end)) : ~0ull;
    const unsigned km = step_mask<BF>(bm);                        // active k-steps of the first layer
    // Bias and head-weight columns wait in LDS: the epilogues then hold no
    // global reads, and their waits leave the next product's prefetched
    // weights in flight (kept in registers, they cost the BF16 form a wave
    // per SIMD).
    constexpr int kVec = N1 + N2 + 2 * N3;                    // b1, b2, b3, w4
    __shared__ __attribute__((aligned(16))) float s_vec[kVec];
    const float *const s_b1 = s_vec, *const s_b2 = s_vec + N1, *const s_b3 = s_b2 + N2, *const s_w4 = s_b3 + N3;
    static_assert(kVec % 4 == 0 && kVec / 4 <= kThreads, "one load per thread");
    const f32x4 vecs = ((const gfloat4*)sp->vec)[min(t, kVec / 4 - 1)];
    __shared__ int s_ob[64];                                  // active adjoint output blocks, then -1
    __shared__ int s_no;
    __shared__ __attribute__((aligned(16))) float s_rinv[TM]; // 1 / the scale of the operand's rows in act
    auto stage_vectors = [&]() {
        if (t < kVec / 4) *(f32x4*)(s_vec + 4 * t) = vecs;
        if (w == NW - 1) {
            const int no_pad = block_list(bm, s_ob, 8);
            if (l == 0) s_no = no_pad;
        }
    };
    // The scale of an atom's row for the next product (FP32 form): each wave
    // puts the largest magnitude of its columns into rmax, and after the
    // barrier that also ends the reads of act every wave takes the largest of
    // the four.  rinv: 1 / scale of this lane's rows in act.
    float rinv[MB], rs[MB];
    auto put_max = [&](const float (&mx)[MB]) {
        if (BF) return;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            float v = fmaxf(mx[mb], shfl_xor(mx[mb], 16));
            v = fmaxf(v, shfl_xor(v, 32));
            if (l < 16) rmax[16 * mb + l][w] = v;
        }
    };
    auto take_scales = [&]() {
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            if (BF) {
                rs[mb] = rinv[mb] = 1.f;
                continue;
            }
            const Pow2 q = pow2_scale(max4(0.f, *(const f32x4*)rmax[16 * mb + lr]));
            rs[mb] = q.s;
            rinv[mb] = q.inv;
            if (w == 0 && l < 16) s_rinv[16 * mb + l] = q.inv;
        }
    };
    // ---------------- layer 1: K0 -> N1 over the active k-steps, A streamed
    // from HBM through LDS (gathered by k-step)
    f32x4 h1[MB][NC1];
    {
        // LPS threads load one k-step of a row, 16 bytes each; TPR threads
        // share a row (SPL steps at once), a thread has RJ rows
        typedef typename std::conditional<BF, u16x8, f32x4>::type vec_t;
        constexpr int kVecN = BF ? 8 : 4, LPS = KS / kVecN;
        constexpr int TPR = kThreads / TM > LPS ? kThreads / TM : LPS, SPL = TPR / LPS, RJ = TM * TPR / kThreads;
        constexpr int kPer = CS / SPL;                        // loads per thread, row and chunk
        const int r0 = t / TPR, sub = (t % TPR) / LPS, ci = kVecN * (t % LPS);
        constexpr int RD = kThreads / TPR;                    // a thread's rows are r0 + RD j
        const int nk = __popc(km);
        constexpr bool kConv = kDir && BF;   // float32 features, rounded as they are read
        const vec_t* src[RJ];
#pragma unroll
        for (int j = 0; j < RJ; ++j) {
            const int row = row0 + r0 + RD * j;
            // padding rows read some atom's features; their results are not stored
            src[j] = (const vec_t*)A.aev + (size_t)(kDir ? max(A.row_atom[row], 0) : row) * (K0 / kVecN * (kConv ? 2 : 1));
        }
        vec_t pre[kPer][RJ];
        // the lowest of the steps left, taken off unless it is the last
        auto take = [](unsigned& left) {
            const int k = __builtin_ctz(left);
            left = left & (left - 1) ? left & (left - 1) : left;
            return k;
        };
        // features of the next SPL steps (the last one again past the end:
        // the position is not used)
        auto fload = [&](unsigned& left, vec_t (&d)[RJ]) {
            int kq = take(left);
#pragma unroll
            for (int k = 1; k < SPL; ++k) {
                const int k1 = take(left);
                kq = sub == k ? k1 : kq;
            }
            const int f = step_feature<BF>(kq, ci);
#pragma unroll
            for (int j = 0; j < RJ; ++j) {
                vec_t v;
                if constexpr (kConv) {
                    const f32x4 *p = (const f32x4*)src[j] + max(f, 0) / 4, lo = p[0], hi = p[1];
                    const bf16x8 c = {(__bf16)lo[0], (__bf16)lo[1], (__bf16)lo[2], (__bf16)lo[3],
                                      (__bf16)hi[0], (__bf16)hi[1], (__bf16)hi[2], (__bf16)hi[3]};
                    v = __builtin_bit_cast(vec_t, c);
                } else {
                    v = src[j][max(f, 0) / kVecN];
                }
                d[j] = f >= 0 ? v : vec_t{};
            }
        };
        unsigned left_a = km;                                 // steps not yet staged
        auto gload = [&]() {
#pragma unroll
            for (int q = 0; q < kPer; ++q) fload(left_a, pre[q]);
        };
        float fs[RJ];   // this thread's rows' scales
        auto sstore = [&](int buf) {
#pragma unroll
            for (int j = 0; j < RJ; ++j)
#pragma unroll
                for (int q = 0; q < kPer; ++q) {
                    uint16_t* dst = smem + buf * NP * kCPlane + (r0 + RD * j) * CLD + (q * SPL + sub) * KS + ci;
                    if constexpr (BF) *(u16x8*)dst = pre[q][j];
                    else put4<BF>(dst, kCPlane, pre[q][j], fs[j]);
                }
        };
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NC1; ++nb) h1[mb][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
        // weight fragments of the e-th active step in ring slot e % RS, loaded
        // PD steps ahead; a chunk spans whole ring turns, so every slot index
        // is known at compile time
        constexpr int PD = ring_ahead<BF>(), RS = ring_turn<BF>();
        static_assert(CS % RS == 0, "a chunk holds whole ring turns");
        WFrag<BF> rb[RS][NC1];
        int blk[NC1];
#pragma unroll
        for (int nb = 0; nb < NC1; ++nb) blk[nb] = w + NW * nb;
        unsigned left_b = km;
        auto loadB = [&](WFrag<BF> (&d)[NC1]) { load_b<BF, kF1, NC1>(wb, blk, take(left_b), d); };
        if (nk > 0) {   // a tile of atoms without neighbours has no active k-step (h1 = CELU(b1))
            gload();
#pragma unroll
            for (int t0 = 0; t0 < PD; ++t0) loadB(rb[t0]);
            stage_vectors();
            if constexpr (!BF) {
                // each row's largest magnitude over every active k-step
                float mx[RJ];
#pragma unroll
                for (int j = 0; j < RJ; ++j) {
                    mx[j] = 0.f;
#pragma unroll
                    for (int q = 0; q < kPer; ++q) mx[j] = max4(mx[j], pre[q][j]);
                }
                constexpr int kAtOnce = 8 / SPL;
                unsigned left = left_a;
                for (int e = CS; e < nk; e += kAtOnce * SPL) {
                    vec_t v[kAtOnce][RJ];
#pragma unroll
                    for (int k = 0; k < kAtOnce; ++k) fload(left, v[k]);
#pragma unroll
                    for (int k = 0; k < kAtOnce; ++k)
#pragma unroll
                        for (int j = 0; j < RJ; ++j) mx[j] = max4(mx[j], v[k][j]);
                }
#pragma unroll
                for (int j = 0; j < RJ; ++j) {
#pragma unroll
                    for (int m = 1; m < TPR; m <<= 1) mx[j] = fmaxf(mx[j], shfl_xor(mx[j], m));
                    const Pow2 q = pow2_scale(mx[j]);
                    fs[j] = q.s;
                    if (t % TPR == 0) s_rinv[r0 + RD * j] = q.inv;
                }
            }
            sstore(0);
        } else {
            stage_vectors();
            if (t < TM) s_rinv[t] = 1.f;
        }
        __syncthreads();
        // whole chunks, the next one staged meanwhile, then the steps left
        // (in a loop of its own: see the ring's note on conditional loads)
        const auto step = [&](const uint16_t* cur, int kq) {
            loadB(rb[(kq + PD) % RS]);
            __builtin_amdgcn_sched_barrier(0);   // keep the prefetches ahead of this step's MFMAs
            Frag<BF> a[MB];
            load_a<BF, MB>(cur, kCPlane, CLD, kq, a);
            mfma_kstep<BF, MB, NC1>(a, rb[kq % RS], h1);
        };
        int c = 0;
        for (; c < nk / CS; ++c) {
            gload();
#pragma unroll
            for (int kq = 0; kq < CS; ++kq) step(smem + (c & 1) * NP * kCPlane, kq);
            sstore((c + 1) & 1);
            __syncthreads();
        }
#pragma unroll
        for (int kq = 0; kq < CS - 1; ++kq) {
            if (kq >= nk % CS) break;
            step(smem + (c & 1) * NP * kCPlane, kq);
        }
    }
    // layer 2's first weight fragments, loaded while the epilogue runs
    BPipe<BF, kF2, NC2> p2;
    p2.start(wb, w);
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) rinv[mb] = BF ? 1.f : s_rinv[16 * mb + lr];
    // hidden layer epilogue: the layer's operand h = CELU(z / scales + b) into
    // act, CELU' kept in z
    auto hidden = [&](auto& z, const float* bias, float iw) {
        constexpr int NCB = sizeof(z[0]) / sizeof(z[0][0]);
        f32x4 h[MB][NCB];
        float mx[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const float sc = rinv[mb] * iw * lane_sign;
            mx[mb] = 0.f;
#pragma unroll
            for (int nb = 0; nb < NCB; ++nb) {
                const f32x4 cb = *(const f32x4*)(bias + 16 * (w + NW * nb) + lc);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const Celu c = celu<BF>(BF ? z[mb][nb][r] + cb[r] : fmaf(z[mb][nb][r], sc * col_sign<BF>(r), cb[r]), A.celu);
                    h[mb][nb][r] = c.h;
                    z[mb][nb][r] = c.d;
                }
                mx[mb] = max4(mx[mb], h[mb][nb]);
            }
        }
        put_max(mx);
        __syncthreads();
        take_scales();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NCB; ++nb)
                put4<BF>(act + (16 * mb + lr) * LD + 16 * (w + NW * nb) + lc, kPlane, h[mb][nb], rs[mb]);
        __syncthreads();
    };
    // adjoint epilogue: d = (z / scales) CELU' (dh), its operand in act
    auto adjoint = [&](auto& d, const auto& dh, float iw) {
        constexpr int NCB = sizeof(d[0]) / sizeof(d[0][0]);
        float mx[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const float sc = rinv[mb] * iw * lane_sign;
            mx[mb] = 0.f;
#pragma unroll
            for (int nb = 0; nb < NCB; ++nb) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    d[mb][nb][r] = (BF ? d[mb][nb][r] : d[mb][nb][r] * (sc * col_sign<BF>(r))) * dh[mb][nb][r];
                mx[mb] = max4(mx[mb], d[mb][nb]);
            }
        }
        put_max(mx);
        __syncthreads();
        take_scales();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NCB; ++nb)
                put4<BF>(act + (16 * mb + lr) * LD + 16 * (w + NW * nb) + lc, kPlane, d[mb][nb], rs[mb]);
        __syncthreads();
    };
    hidden(h1, s_b1, iw1);
    // ---------------- layer 2: N1 -> N2
    f32x4 h2[MB][NC2];
    gemm_run<BF, MB>(act, kPlane, wb, p2, h2);
    BPipe<BF, kF3, NC2> p3;
    p3.start(wb, w);
    hidden(h2, s_b2, iw2);
    // ---------------- layer 3: N2 -> N3 (160 padded to 192), head, d3
    BPipe<BF, kA3, NC2> pa3;
    {
        f32x4 z3[MB][NC2];
        gemm_run<BF, MB>(act, kPlane, wb, p3, z3);
        if (A.g_out) pa3.start(wb, w);
        float mx[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const float sc = rinv[mb] * iw3 * lane_sign;
            float part = 0.f;
            mx[mb] = 0.f;
#pragma unroll
            for (int nb = 0; nb < NC2; ++nb) {
                const f32x4 cb = *(const f32x4*)(s_b3 + 16 * (w + NW * nb) + lc);
                const f32x4 cw = *(const f32x4*)(s_w4 + 16 * (w + NW * nb) + lc);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float wc = cw[r];
                    const Celu c = celu<BF>(BF ? z3[mb][nb][r] + cb[r] : fmaf(z3[mb][nb][r], sc * col_sign<BF>(r), cb[r]), A.celu);
                    part += c.h * wc;
                    z3[mb][nb][r] = wc * c.d;
                }
                mx[mb] = max4(mx[mb], z3[mb][nb]);
            }
            // the four lanes that share a row (columns), fixed butterfly
            part += shfl_xor(part, 16);
            part += shfl_xor(part, 32);
            if (l < 16) epart[16 * mb + l][w] = part;
        }
        put_max(mx);
        __syncthreads();
        take_scales();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int nb = 0; nb < NC2; ++nb)
                put4<BF>(act + (16 * mb + lr) * LD + 16 * (w + NW * nb) + lc, kPlane, z3[mb][nb], rs[mb]);
    }
    if (t < TM) {
        const float e = ((epart[t][0] + epart[t][1]) + (epart[t][2] + epart[t][3])) + hb4;
        const int row = row0 + t;
        if (kEns) {
            A.E_net[(size_t)net * A.rows + row] = e;
        } else {
            A.E_row[row] = e;
            const int a = A.row_atom[row];
            if (a >= 0 && A.E_atomo) A.E_atomo[a] = e;
        }
    }
    if (!A.g_out) return;
    __syncthreads();
    // ---------------- adjoint 3: d2 = (W3^T d3) * CELU'(h2)
    BPipe<BF, kA2, NC1> pa2;
    {
        f32x4 d[MB][NC2];
        gemm_run<BF, MB>(act, kPlane, wb, pa3, d);
        pa2.start(wb, w);
        adjoint(d, h2, ia3);
    }
    // ---------------- adjoint 2: d1 = (W2^T d2) * CELU'(h1)
    // adjoint 1 runs over the active output blocks (16 columns each, listed
    // in s_ob and padded with -1 to a multiple of eight): passes of sixteen
    // blocks, then one of eight for a remainder, dealt evenly to the waves
    constexpr int NG = 16 / NW, NGR = 8 / NW;
    const int no = __builtin_amdgcn_readfirstlane(s_no), n16 = no / 16;
    BPipe<BF, kA1, NG> pg;
    BPipe<BF, kA1, NGR> pr;
    {
        f32x4 d[MB][NC1];
        gemm_run<BF, MB>(act, kPlane, wb, pa2, d);
        if (!kEns) {
            if (n16 > 0) pg.start(wb, s_ob + NG * w);
            else if (no > 0) pr.start(wb, s_ob + NGR * w);
        }
        adjoint(d, h1, ia2);
    }
    if (kEns) {
        // d1 tile out (this network's slice); the first layer's adjoint sums over networks
        u16x8* dst = (u16x8*)(A.d1_out + ((size_t)net * A.rows + row0) * NP * N1);
        for (int q = t; q < TM * NP * N1 / 8; q += kThreads) {
            const int row = q / (NP * N1 / 8), c = q % (NP * N1 / 8), p = c / (N1 / 8);
            dst[q] = *(const u16x8*)(act + p * kPlane + row * LD + 8 * (c % (N1 / 8)));
        }
        if (!BF && w == 0 && l < 16)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) A.d1_inv[(size_t)net * A.rows + row0 + 16 * mb + l] = rinv[mb];
        return;
    }
    // ---------------- adjoint 1: g = W1^T d1 over the active output blocks
    __shared__ float s_gs[TM];
    __shared__ int s_row[TM];
    if (t < TM) {
        s_gs[t] = BF ? 1.f : s_rinv[t] * ia1;
        s_row[t] = kDir ? A.row_atom[row0 + t] : row0 + t;
    }
    __syncthreads();
    const auto row_of = [&](int i) { return s_row[i]; };
    for (int pass = 0; pass < n16; ++pass) {
        const int* ob = s_ob + 16 * pass + NG * w;
        f32x4 gacc[MB][NG];
        gemm_run<BF, MB>(act, kPlane, wb, pg, gacc);
        pg.start(wb, s_ob + 16 * min(pass + 1, n16 - 1) + NG * w);
        store_g<BF, MB, NG>(A.g_out, row_of, gacc, ob, s_gs);
    }
    if (no > 16 * n16) {
        if (n16 > 0) pr.start(wb, s_ob + 16 * n16 + NGR * w);
        f32x4 gacc[MB][NGR];
        gemm_run<BF, MB>(act, kPlane, wb, pr, gacc);
        store_g<BF, MB, NGR>(A.g_out, row_of, gacc, s_ob + 16 * n16 + NGR * w, s_gs);
    }
}

// Ensemble, first layer's adjoint summed over networks:
//   g = (1 / n_nets) sum_net W1_net^T d1_net
// and the ensemble-mean energies.  Block (tile, pass): the tile's active
// sixteen output blocks of the pass (as in the single-network kernel).  FP32
// form: each network's product has its own scales, and is added to the sum
// in float32; BF16: one accumulation over K = 256 n_nets.
template <bool BF, int TM, bool kDir>
__global__ __launch_bounds__(kThreads, BF ? 2 : 3) void k_ens_adj1(const FusedArgs A, int n_nets, float inv_nets,
                                                                  float* E_atom_net, int n_atoms) {
    constexpr int NG = 16 / NW;
    constexpr int NP = planes<BF>();
    constexpr int MB = TM / 16;
    constexpr int kPlane = TM * LD;
    __shared__ __attribute__((aligned(16))) uint16_t act[NP * kPlane];
    const int row0 = xcd_tile((A.rows + TM - 1) / TM) * TM, pass = blockIdx.y;
    if (row0 >= A.rows) return;
    const int s = tile_species_of(A.meta, row0), row_end = segment_end(A.meta, s);
    if (row0 >= row_end) return;
    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t / kWave), l = lane_id();
    __shared__ int s_ob[64];
    __shared__ int s_no;
    if (t < kWave) {
        const unsigned long long bm = A.amask ? species_blocks(tile_species<TM>(A.amask, row0, row_end)) : ~0ull;
        const int no = block_list(bm, s_ob, 16);
        if (l == 0) s_no = no;
    }
    __syncthreads();
    const bool work = A.g_out && 16 * pass < s_no;   // block-uniform
    const int* ob = s_ob + 16 * pass + NG * w;
    f32x4 acc[MB][NG];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NG; ++nb) acc[mb][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int net = 0; work && net < n_nets; ++net) {
        const FusedNet::Species* __restrict__ sp = &A.nets[net].sp[s];
        const PackBuf wb = pack_buf<BF>(sp->packs);
        BPipe<BF, kA1, NG> p;
        p.start(wb, ob);
        const u16x8* src = (const u16x8*)(A.d1_out + ((size_t)net * A.rows + row0) * NP * N1);
        for (int q = t; q < TM * NP * N1 / 8; q += kThreads) {
            const int row = q / (NP * N1 / 8), c = q % (NP * N1 / 8), pl = c / (N1 / 8);
            *(u16x8*)(act + pl * kPlane + row * LD + 8 * (c % (N1 / 8))) = src[q];
        }
        __syncthreads();
        if constexpr (BF) {
            gemm_run<BF, MB, kA1, NG, false>(act, kPlane, wb, p, acc);
        } else {
            f32x4 d[MB][NG];
            gemm_run<BF, MB>(act, kPlane, wb, p, d);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                const f32x4 sc = *(const f32x4*)(A.d1_inv + (size_t)net * A.rows + row0 + 16 * mb + 4 * (l >> 4)) *
                                 sp->inv[kA1];
#pragma unroll
                for (int nb = 0; nb < NG; ++nb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[mb][nb][r] = fmaf(d[mb][nb][r], sc[r], acc[mb][nb][r]);
            }
        }
        __syncthreads();
    }
    if (work) {
        __shared__ float s_gs[TM];
        __shared__ int s_row[TM];
        if (t < TM) {
            s_gs[t] = inv_nets;
            s_row[t] = kDir ? A.row_atom[row0 + t] : row0 + t;
        }
        __syncthreads();
        store_g<BF, MB, NG>(A.g_out, [&](int i) { return s_row[i]; }, acc, ob, s_gs);
    }
    if (pass == 0 && t < TM) {
        const int row = row0 + t;
        float e = 0.f;
        for (int net = 0; net < n_nets; ++net) e += A.E_net[(size_t)net * A.rows + row];
        e *= inv_nets;
        A.E_row[row] = e;
        const int a = A.row_atom[row];
        if (a >= 0) {
            if (A.E_atomo) A.E_atomo[a] = e;
            if (E_atom_net)
                for (int net = 0; net < n_nets; ++net)
                    E_atom_net[(size_t)net * n_atoms + a] = A.E_net[(size_t)net * A.rows + row];
        }
    }
}

}  // namespace

// ---------------------------------------------------------------- host side

bool fused_mlp_shape(const int* widths, int n_layers, int ns) {
    const int dim = ns * kNr + ns * (ns + 1) / 2 * kNa * kNz;
    return n_layers == 4 && dim <= K0 && dim > K0 - 64 && widths[1] == N1 && widths[2] == N2 &&
           widths[3] <= N3 && widths[3] > N3 - 64 && widths[4] == 1;
}

static uint16_t host_f16_bits(float f) {   // nearest even; |f| below the float16 range's end
    uint32_t u;
    std::memcpy(&u, &f, 4);
    const uint32_t sign = (u >> 16) & 0x8000u, a = u & 0x7fffffffu;
    if (a >= 255u << 23) return (uint16_t)(sign | 0x7c00u | (a > 255u << 23 ? 0x200u : 0u));
    if (a >= 113u << 23) return (uint16_t)(sign | (((a + 0xfffu + ((a >> 13) & 1u)) >> 13) - (112u << 10)));
    const uint32_t sh = 126u - (a >> 23);   // below 2^-14: whole numbers of 2^-24
    if (sh > 24) return (uint16_t)sign;
    const uint32_t m = (a & 0x7fffffu) | 0x800000u, q = m >> sh, rem = m & ((1u << sh) - 1), half = 1u << (sh - 1);
    return (uint16_t)(sign | (q + (rem > half || (rem == half && (q & 1u)))));
}

static float host_f16_value(uint16_t h) {
    const uint32_t e = (h >> 10) & 31u, m = h & 0x3ffu;
    if (e == 31) return m ? NAN : (h & 0x8000u ? -INFINITY : INFINITY);
    if (e == 0) return (h & 0x8000u ? -1.f : 1.f) * (float)m * (1.f / 16777216.f);
    const uint32_t u = ((uint32_t)(h & 0x8000u) << 16) | ((e + 112u) << 23) | (m << 13);
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

uint16_t host_bf16_bits(float f);

// Packs B[k][n] (k < K, n < N, accessor) into MFMA fragment order; fragment
// nb K/32 + ks (column block nb, k-step ks) holds plane p at [p][lane][e]
// (16-bit values), then the remainders' four bits each (remainders()) at [lane],
// of B[32 ks + 8 (lane/16) + e][16 nb + lane%16] (BF16: the rounded value; FP32
// form: hi and lo float16 of s B times the columns' signs).
//
// hi + lo holds 23 of a weight's 24 bits: for one weight in four, what hi leaves
// lies halfway between two float16 numbers.  The remainder, a power of two,
// completes the weight: lo is the lower of the two at even e and the upper at
// odd e, so that the remainders, of which an accumulator's last bits drop a
// part, are as often negative as positive.  (Left out, these errors, the same
// for every atom, made the mean error of a species' energies 6.1e-9 of their
// terms over six sets of weights, the largest 1.7e-8; with the remainders
// 4.4e-9 and 1.0e-8; float32 MFMAs 4.3e-9 and 1.3e-8.)
template <typename F>
static void pack_matrix(char* out, bool bf16, float s, int K, int N, F B) {
    for (int n = 0; n < N; ++n) {
        for (int k = 0; k < K; ++k) {
            const float v = bf16 ? B(k, n) : B(k, n) * col_sign<false>(n);
            const size_t frag = (size_t)(n / 16) * (K / KS) + k / KS;
            const int lane = (k % KS) / 8 * 16 + n % 16, e = k % 8;
            if (bf16) {
                ((uint16_t*)(out + frag * frag_bytes<true>()))[lane * 8 + e] = host_bf16_bits(v);
                continue;
            }
            uint16_t* planes = (uint16_t*)(out + frag * frag_bytes<false>());
            const uint16_t hi = host_f16_bits(v * s);
            const float left = v * s - host_f16_value(hi);
            uint16_t lo = host_f16_bits(left);
            if (host_f16_value(lo) != left) {
                // the neighbour of left that leaves a remainder of e's sign
                const bool above = host_f16_value(lo) > left, up = e & 1;
                const uint16_t to = above == up ? lo : (lo & 0x8000u) ? (up ? lo - 1 : lo + 1) : (up ? lo + 1 : lo - 1);
                const float rest = fabsf(left - host_f16_value(to)) * kRest;
                if (rest >= 0x1p-14f && rest <= 1.f) {
                    const int f = ilogbf(rest) + 15;
                    if (ldexpf(1.f, f - 15) == rest) {
                        lo = to;
                        const uint64_t bits = (uint64_t)f << rest_bit(e);
                        ((uint32_t*)(planes + 1024))[lane] |= (uint32_t)(bits | bits >> 32);
                    }
                }
            }
            planes[lane * 8 + e] = hi;
            planes[512 + lane * 8 + e] = lo;
        }
    }
}

// Builds the six packs of one species from row-major W_l [out][in] (host) at
// zeroed dst; inv: 1 / the scale of each.  Returns bytes used at dst (dst may be
// null to size).
size_t pack_fused_species(char* dst, float* inv, bool bf16, const float* W1, const float* W2, const float* W3,
                          int n_in, int n3) {
    const size_t unit = bf16 ? frag_bytes<true>() : frag_bytes<false>();
    if (!dst) return pack_first(kPacks) * unit;
    // logical padded matrices: W1p [N1][K0], W2p [N2][N1], W3p [N3][N2] (rows >= n3 zero)
    auto w1 = [&](int o, int i) { return i >= 0 && i < n_in ? W1[(size_t)o * n_in + i] : 0.f; };
    auto w2 = [&](int o, int i) { return W2[(size_t)o * N1 + i]; };
    auto w3 = [&](int o, int i) { return o < n3 ? W3[(size_t)o * N2 + i] : 0.f; };
    auto largest = [](const float* W, size_t n) {
        float m = 0.f;
        for (size_t k = 0; k < n; ++k) m = W[k] > m ? W[k] : (-W[k] > m ? -W[k] : m);
        return m;
    };
    Pow2 sc[3] = {{1.f, 1.f}, {1.f, 1.f}, {1.f, 1.f}};
    if (!bf16) {
        sc[0] = pow2_scale(largest(W1, (size_t)N1 * n_in));
        sc[1] = pow2_scale(largest(W2, (size_t)N2 * N1));
        sc[2] = pow2_scale(largest(W3, (size_t)n3 * N2));
    }
    for (int q = 0; q < kPacks; ++q) {
        auto B = [&](int k, int n) -> float {
            switch (q) {
                case kF1:   // forward: B[k][n] = W[n][k]
                    return w1(n, bf16 ? step_feature<true>(k / KS, k % KS) : step_feature<false>(k / KS, k % KS));
                case kF2: return w2(n, k);
                case kF3: return w3(n, k);
                case kA3: return w3(k, n);   // adjoint: B[k][n] = W[k][n]
                case kA2: return w2(k, n);
                default: return w1(k, n);
            }
        };
        const Pow2& c = sc[q < 3 ? q : 5 - q];
        pack_matrix(dst + pack_first(q) * unit, bf16, c.s, kPackK[q], kPackN[q], B);
        inv[q] = c.inv;
    }
    return pack_first(kPacks) * unit;
}

size_t fused_net_bytes() { return sizeof(FusedNet); }

// Ensembles run as the two-kernel split (every network's forward and adjoint
// down to d1, then the first-layer adjoint summed over networks).  For one
// network the split measured within a few per cent of the fused kernel at
// 2,048-8,192 atoms (and slower in BF16), so a single network stays fused.
bool mlp_split(const nnp_model* m, int n_atoms) {
    (void)n_atoms;
    return m->fused && m->n_nets > 1;
}

// Fills the device-table entry of one network (host copy) from each species'
// packs, their inverse scales and the bias and head columns.
void fused_net_entry(void* out, int ns, const char* const* packs, const float (*inv)[kFusedPacks],
                     const float* const* vec, const float* b4) {
    FusedNet& E = *(FusedNet*)out;
    std::memset(&E, 0, sizeof(E));
    for (int q = 0; q < ns; ++q) {
        E.sp[q].packs = packs[q];
        E.sp[q].vec = vec[q];
        for (int k = 0; k < kPacks; ++k) E.sp[q].inv[k] = inv[q][k];
        E.sp[q].b4 = b4[q];
    }
}

namespace {

// Tile height.  A tile streams its species' whole weight packs whatever its
// height, so 32 rows are the rule as soon as one network's 16-row tiles would
// outnumber the CUs; below that a tile is alone on its CU, and the shorter one
// ends sooner.  FP32, us with 16 and with 32 rows: a 19-atom molecule 31 and 42
// (on an idle card), 3,000 water atoms 22.1 and 26.3, dense organic ones 54 and
// 63; 4,500 27.3 and 26.5, 70 and 67; 9,000 38 and 36, 103 and 96.  An
// ensemble's grid holds its networks' tiles side by side, so that 32 rows would
// pay from fewer atoms (eight networks: 77 and 84 at 900 water atoms, 119 and 114
// at 3,000; organic 133 and 114, 255 and 188); its line is the single network's.
// The BF16 form keeps its 12 Ki atoms, and its ensemble takes 64 rows from 48 Ki
// atoms, where the first-layer adjoint over all networks gains from it.
int fused_tile_rows(int n_atoms, bool bf, bool ens) {
    if (!bf) return n_atoms >= 4096 ? 32 : 16;
    return n_atoms >= 48 * 1024 && ens ? 64 : (n_atoms >= 12 * 1024 ? 32 : 16);
}

FusedArgs fused_args(const nnp_model* m, const MlpWs& W, const void* aev, float* g_out, float* E_row, float* E_atomo) {
    const bool bf = m->precision == NNP_BF16_MLP;
    FusedArgs A;
    std::memset(&A, 0, sizeof(A));
    A.nets = (const FusedNet*)(bf ? m->fused_tab_bf16 : m->fused_tab_fp32);
    A.meta = W.meta;
    A.row_atom = W.row_atom;
    A.aev = aev;
    A.g_out = g_out;
    A.E_row = E_row;
    A.E_atomo = E_atomo;
    const double k = 1.4426950408889634 / (double)m->celu_alpha;
    float k_hi = (float)k;
    if ((double)k_hi >= k) k_hi = nextafterf(k_hi, 0.f);
    A.celu = {m->celu_alpha, 1.f / m->celu_alpha, k_hi, (float)(k - (double)k_hi)};
    A.rows = W.rows_max;
    A.amask = W.amask;
    return A;
}

}  // namespace

namespace {

template <bool BF, int TM>
void run_fused(const FusedArgs& A, bool direct, int grid, hipStream_t s) {
    if (direct) k_mlp_fused<BF, TM, false, true><<<grid, kThreads, 0, s>>>(A);
    else k_mlp_fused<BF, TM, false, false><<<grid, kThreads, 0, s>>>(A);
}

template <bool BF, int TM, bool kDir>
void run_ensemble(const FusedArgs& A, dim3 front, dim3 adj1, int n_nets, float inv, float* E_atom_net, int n_atoms,
                  hipStream_t s) {
    k_mlp_fused<BF, TM, true, kDir><<<front, kThreads, 0, s>>>(A);
    k_ens_adj1<BF, TM, kDir><<<adj1, kThreads, 0, s>>>(A, n_nets, inv, E_atom_net, n_atoms);
}

}  // namespace

hipError_t launch_mlp_fused(const nnp_model* m, const MlpWs& W, const void* aev, float* g_out, bool direct,
                            float* E_row, float* E_atomo, int n_atoms, hipStream_t s) {
    const bool bf = m->precision == NNP_BF16_MLP;
    const FusedArgs A = fused_args(m, W, aev, g_out, E_row, E_atomo);
    const int tm = fused_tile_rows(n_atoms, bf, false);
    const int grid = ceil_div(ceil_div(W.rows_max, tm), kXcds) * kXcds;   // whole rounds of the XCDs (xcd_tile)
    if (bf) {
        if (tm == 32) run_fused<true, 32>(A, direct, grid, s);
        else run_fused<true, 16>(A, direct, grid, s);
    } else {
        if (tm == 32) run_fused<false, 32>(A, direct, grid, s);
        else run_fused<false, 16>(A, direct, grid, s);
    }
    return hipGetLastError();
}

// Ensemble of m->n_nets networks on the shared features: every network's
// forward and adjoint down to d1 (grid.y = network), then the first layer's
// adjoint summed over networks and the mean energies.  d1_scratch:
// [n_nets][rows_max][256] (float32-sized), d1_inv and E_net: [n_nets][rows_max];
// E_atom_net: [n_nets][n_atoms] per-network atomic energies or null.
hipError_t launch_mlp_ensemble(const nnp_model* m, const MlpWs& W, const void* aev, float* g_out, bool direct,
                               float* E_row, float* E_atomo, int n_atoms, void* d1_scratch, float* d1_inv,
                               float* E_net, float* E_atom_net, hipStream_t s) {
    const bool bf = m->precision == NNP_BF16_MLP;
    FusedArgs A = fused_args(m, W, aev, g_out, E_row, E_atomo);
    A.d1_out = (uint16_t*)d1_scratch;
    A.d1_inv = d1_inv;
    A.E_net = E_net;
    const int tm = fused_tile_rows(n_atoms, bf, true);
    const int gx = ceil_div(ceil_div(W.rows_max, tm), kXcds) * kXcds;   // whole rounds of the XCDs (xcd_tile)
    const dim3 g1(gx, m->n_nets), g2(gx, g_out ? 4 : 1);
    const float inv = 1.f / (float)m->n_nets;
    const auto run = [&](auto grouped, auto dir) {
        (direct ? dir : grouped)(A, g1, g2, m->n_nets, inv, E_atom_net, n_atoms, s);
    };
    if (bf) {
        if (tm == 64) run(run_ensemble<true, 64, false>, run_ensemble<true, 64, true>);
        else if (tm == 32) run(run_ensemble<true, 32, false>, run_ensemble<true, 32, true>);
        else run(run_ensemble<true, 16, false>, run_ensemble<true, 16, true>);
    } else {
        if (tm == 32) run(run_ensemble<false, 32, false>, run_ensemble<false, 32, true>);
        else run(run_ensemble<false, 16, false>, run_ensemble<false, 16, true>);
    }
    return hipGetLastError();
}

}  // namespace nnp
