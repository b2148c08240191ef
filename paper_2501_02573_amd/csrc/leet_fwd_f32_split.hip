// Chunk-walk kernel for fp32 inputs of width 128 (gfx950): fp32 products on the bf16 matrix instructions.
//
// Same algorithm as the wide 16-bit kernel: one workgroup per segment of a (batch, head) sequence
// walks the tokens in order (Alg. 2, Appendix B.2, with the decaying mask of Eq. "BCMV" and the
// weight split of Alg. 4, Appendix B.3), here in tiles of L = 32 tokens:
//
//     O_t     = ((Q_t K_t^T) .* D) V_t + Lam (Q_t S_t)       D[i][j] = gamma^(i-j), i >= j
//     S_{t+1} = gamma^L S_t + (Gam K_t)^T V_t                Lam = diag(gamma^(i+1)), Gam = diag(gamma^(L-1-j))
//
// The fp32 matrix instructions run at a sixteenth of the bf16 rate, and a kernel built on them is
// bound by their issue.  Here every fp32 operand x is written as x0 + x1 + x2 with bf16 terms, each the
// upper 16 bits of what the terms before it leave: 8 + 8 + 8 significant bits hold all 24 of x, and bf16
// has the exponent range of fp32, so the sum is exactly x.  A product needs all partial products
// but a2 b2, which is below 2^-32 of it: left out, a1 b2 and a2 b1 make one product in itself (a token's first
// P V, one-hot q and k) wrong by up to 2^-22.  Each partial product is exact in fp32 and the sums are
// fp32 accumulators as before, with fewer roundings (one instruction contracts 16 or 32 terms, not 4):
// eight instructions at 16 times the rate.
//
// Range: the bf16 matrix instructions take denormal terms and sums (below 2^-126) as zero, and an infinity leaves
// x - x0 = NaN.  So the walk watches the smallest nonzero operands and whether its results are finite, and where
// something is out of range the segment is walked again with fp32 matrix instructions (walk_fp32), whose
// results stand for every operand.  Ordinary data never does that (nor zeros behind a sequence: B4 H16 N4096 261 us, half of it
// zeros 247; all out of range 325, an infinity in one sequence 344 to 441 by its place); the watching costs some 60 of 650 vector
// operations a tile (B4 H16 N4096, before the walk overlapped them with MFMAs, 273 -> 282 us; without it q, k ~ 2^-60 with v ~ 2^104
// came out with errors of 6e-4).
//
// Work split: a column tile of 32 value columns belongs to two waves (in the pre-pass: one),
// which hold half of the key dimension each: S[half of dk][cols] in fp32 accumulators for the whole walk.
// Each computes its half of the sum Q S and the scores' product with one half of the keys; the two sums
// meet in LDS on their way out.  Eight waves, one workgroup a compute unit; in the pre-pass four and two (whose
// phases overlap by themselves).
//
// What bounds it: the power of its matrix and vector instructions.  Per 32-token tile there are 624 MFMAs of 32 cycles (of 4
// SIMDs) and, per wave, some 650 vector operations, most of them splits.  The walk forms an operand while an MFMA that does not
// need it is running: the next tile's k and q during G4, Gam V during G3, the state's update during G2; each wave of a pair
// splits its half of V and hands the weighted half to the other through LDS.  Two barriers a tile.  B4 H16 N4096, walk: 349
// thousand cycles with the phases one after the other and three barriers, 307 so (313 with the range looked up every second
// tile); 183 -> 171 us at the clock of a first
// run.  In a steady run the clock gives way (2.0 -> 1.6 GHz) and a call gains less, 266 -> 254 us; B9 H33 N2000 611 -> 553,
// B16 H32 N300 122 -> 116.  Before that, against fp32 MFMAs: 319 -> 282, B1 H32 N777 53.5 -> 45.9
// (walk_fp32 alone, B1 H300 N2000: 805, here 630).
// Against 64 bits a single product errs by at most 5.99e-8 of itself (5.95e-8 with fp32 MFMAs).  Sums round less
// often: outputs err 0.30 to 0.47 and states 0.33 to 0.83 as much as with fp32 MFMAs, in the 2-norm over forty sizes; over forty
// drawn ones (2 to 8000 tokens, with and without decay and entering state) outputs 0.63e-7 to 1.74e-7, states 0.30e-7 to
// 2.28e-7.  The largest single error of a state after two tokens, in units of its rms and over 200 seeds, is 4.2e-7 on
// average (5.3e-7) and 8.4e-7 at worst (6.7e-7).
//
// MFMA conventions: an A (B) operand of 32x32x16 (16x16x32) holds, in lane l, row (column) l%32
// (l%16) and eight contraction slots of group l/32 (l/16); a 32x32 (16x16) accumulator holds column
// l%32 (l%16) and, in register r, row 8(r/4) + 4(l/32) + r%4 (row 4(l/16) + r).  A contraction may
// assign indices to slots in any way, as long as A and B agree.
//
//   G1  P^T[j][i]  = sum_dk K[j][dk] Q[i][dk]     three 16x16 tiles (it >= jt), by waves 0, 1 and 2;
//                                                 accumulator row 4q + r of a tile is key j = 16jt + q + 4r
//       P^T       *= D^T                          then split and handed to all waves as P[i][slot],
//                                                 slot 16jt + 4q + r
//   G3  O[i][c]    = sum_dk Q[i][dk] S[dk][c]     A = Q rows, B = S accumulators, split in registers
//       O         *= gamma^(i+1)
//   G2  O[i][c]   += sum_j P[i][j] V[j][c]        A = P rows, B = V, straight from global memory into
//                                                 registers in slot order (a wave's columns are its own)
//   G4  S[dk][c]  += sum_j K^T[dk][j] (Gam V)[j][c]   A = K through transposing LDS reads
//                                                 (ds_read_b64_tr_b16), B = the V registers times Gam
// Slots of 16 keys run 0 4 8 12, 1 5 9 13, ...: a transposing read then touches rows four apart,
// which the padded rows spread over all LDS banks.  G4 assigns key-dimension index dk = 32t + pi(m)
// to accumulator row m (pi swaps bits 2 and 3), so that registers 8h..8h+7 of S hold the eight
// consecutive dk that one 16-byte Q read contracts with.
// O accumulators are columns across lanes: a store instruction writes two whole 128-byte row pieces.
//
// A ragged last tile (L < 32) is left-aligned and zero below its tokens: all weights stay valid but
// Gam = gamma^(L-1-j), and gamma^L.
#include "leet_common.hpp"

namespace leet {

namespace f32s {

constexpr int D = 128;     // width of q, k, v and out rows
constexpr int kTile = 32;  // tokens per step of the walk

// The waves of a column tile: two share the key dimension, except in the pre-pass.
constexpr int parts(bool out) { return out ? 2 : 1; }
constexpr int threads(bool out) { return D / 32 * parts(out) * 64; }

typedef short s16x4 __attribute__((ext_vector_type(4)));

// The pre-pass (kOut = false) reads no Q and forms no scores; one barrier a tile.
template <bool kOut>
struct Smem {
    static constexpr int RS = D + 8;    // padded row strides (elements)
    static constexpr int RP = kTile + 8;
    static constexpr int RO = kTile + 8;  // output scratch of a wave (floats)
    uint16_t k[2][3 * kTile * RS];   // three planes each; this tile's and the next one's
    uint16_t q[kOut ? 3 * kTile * RS : 8];
    u32x4 gv[kOut ? 2 * (D / 32) : 1][3][64];   // Gam V of a wave's half of the keys, as operand
    uint16_t p[kOut ? 3 * kTile * RP : 8];      // masked scores P[i][slot]
    float o[kOut ? 2 * (D / 32) * kTile * RO : 4];  // output tiles of the waves
    float lw[kTile];       // gamma^(i+1)
    float gw[2][kTile];    // gamma^(31-j) in slot order; gamma^(L-1-j) of the segment's last tile
    float pw[kTile + 4];   // gamma^n, n = 0..32
    int bad[2];            // out of range: seen so far, in the whole walk
};

// The smallest magnitude of kN values; and of those other than zero, as twice its bits minus one, which puts zero
// above everything else.  The first is half an operation a value and enough for data without zeros.
template <int kN, class Get>
__device__ __forceinline__ float smallest(Get x) {
    float m = __builtin_fabsf(x(0));
#pragma unroll
    for (int i = 1; i < kN; ++i) m = __builtin_fminf(m, __builtin_fabsf(x(i)));
    return m;
}
__device__ __forceinline__ uint32_t rank_nonzero(float x) { return (__float_as_uint(x) << 1) - 1; }
template <int kN, class Get>
__device__ __forceinline__ uint32_t smallest_nonzero(Get x) {
    uint32_t m = ~0u;
#pragma unroll
    for (int i = 0; i < kN; ++i) m = min(m, rank_nonzero(x(i)));
    return m;
}
// Whether one of them is nonzero and below `least`.
template <int kN, class Get>
__device__ __forceinline__ bool has_small(Get x, float least) {
    return __any(smallest<kN>(x) < least) ? smallest_nonzero<kN>(x) < rank_nonzero(least) : false;
}
// 2^e as a float, -126 <= e <= 127
__device__ __forceinline__ float pow2(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }
// exponent of the largest of four values; 0 where that is zero, denormal or not finite
__device__ __forceinline__ int exponent4(const float* x) {
    const uint32_t a = __float_as_uint(x[0]) << 1, b = __float_as_uint(x[1]) << 1, c = __float_as_uint(x[2]) << 1, d = __float_as_uint(x[3]) << 1;
    const int e = (int)(max(max(a, b), max(c, d)) >> 24);
    return e == 0 || e == 255 ? 0 : e - 127;
}

// an operand as three bf16 terms
struct Frag3 {
    u32x4 x[3];
};

// Two values -> their three terms, each packed in a pair.
struct Pair3 {
    uint32_t x[3];
};
__device__ __forceinline__ Pair3 split2(float a, float b) {
#pragma clang fp contract(off)
    auto upper = [](float lo, float hi) { return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u); };
    auto rest = [](float x) { return x - __uint_as_float(__float_as_uint(x) & 0xffff0000u); };
    Pair3 s;
    s.x[0] = upper(a, b);
    const float ra = rest(a), rb = rest(b);
    s.x[1] = upper(ra, rb);
    s.x[2] = upper(rest(ra), rest(rb));
    return s;
}

// words 2e and 2e+1 of an operand
__device__ __forceinline__ void put2(Frag3& f, int e, float a, float b) {
    const Pair3 s = split2(a, b);
#pragma unroll
    for (int i = 0; i < 3; ++i) f.x[i][e] = s.x[i];
}

// four consecutive values -> 8 bytes of each of the three planes (plane stride `plane` elements)
__device__ __forceinline__ void store4(uint16_t* dst, int plane, float a, float b, float c, float d) {
    const Pair3 lo = split2(a, b), hi = split2(c, d);
#pragma unroll
    for (int i = 0; i < 3; ++i) *reinterpret_cast<u32x2*>(dst + i * plane) = u32x2{lo.x[i], hi.x[i]};
}

// The seven partial products below the leading one; they have an accumulator of their own, so that
// their roundings are 2^-6 of the sum's and only the leading product and one addition round at full size.
__device__ __forceinline__ f32x16 mma32_small(const Frag3& a, const Frag3& b, f32x16 c) {
    c = ElemBf16::mfma32(a.x[1], b.x[2], c);
    c = ElemBf16::mfma32(a.x[2], b.x[1], c);
    c = ElemBf16::mfma32(a.x[2], b.x[0], c);
    c = ElemBf16::mfma32(a.x[0], b.x[2], c);
    c = ElemBf16::mfma32(a.x[1], b.x[1], c);
    c = ElemBf16::mfma32(a.x[1], b.x[0], c);
    return ElemBf16::mfma32(a.x[0], b.x[1], c);
}

__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mma16_small(const Frag3& a, const Frag3& b, f32x4 c) {
    c = mfma16(a.x[1], b.x[2], c);
    c = mfma16(a.x[2], b.x[1], c);
    c = mfma16(a.x[2], b.x[0], c);
    c = mfma16(a.x[0], b.x[2], c);
    c = mfma16(a.x[1], b.x[1], c);
    c = mfma16(a.x[1], b.x[0], c);
    return mfma16(a.x[0], b.x[1], c);
}

// ds_read_b64_tr_b16: within each group of 16 lanes, lane i receives element i%4 of
// the 8-byte rows addressed by lanes i/4, 4+i/4, 8+i/4, 12+i/4 of the group.
__device__ __forceinline__ u32x2 lds_tr(const uint16_t* p) {
    s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4*)(const_cast<uint16_t*>(p)));
    return __builtin_bit_cast(u32x2, r);
}

// The scheduler's order for a region: an MFMA, then kValu vector operations and what LDS work there is, kMfma times.
template <int kMfma, int kValu>
__device__ __forceinline__ void interleave() {
#pragma unroll
    for (int i = 0; i < kMfma; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, kValu, 0);
        __builtin_amdgcn_sched_group_barrier(0x80, 1, 0);
    }
}

// The tile of tokens tok0 .. min(tok0 + 31, tok_end - 1) of a tensor with rows of D floats (none if tok0 >= tok_end).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const float* base, int tok0, int tok_end) {
    // all of it is the same in every lane; the compiler is told, since it moves part of the arithmetic to vector registers
    const uintptr_t addr = reinterpret_cast<uintptr_t>(base) + (size_t)tok0 * (D * 4);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)addr), hi = __builtin_amdgcn_readfirstlane((uint32_t)(addr >> 32));
    const int bytes = __builtin_amdgcn_readfirstlane(max(min(kTile, tok_end - tok0), 0) * (D * 4));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(((uintptr_t)hi << 32) | lo), 0, bytes, 0x00027000);
}
// kStream: with the nontemporal hint
template <bool kStream>
__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kStream ? 2 : 0));
}
__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t r, int off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
// nontemporal: the output is written once and not read again here
__device__ __forceinline__ void store4_nt(f32x4 x, __amdgpu_buffer_rsrc_t r, int off) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), r, off, 0, 2);
}

}  // namespace f32s

// kOut = true : full walk (outputs + state).   kOut = false : state only (segment pre-pass).
// kStream: q, k, v exceed the last-level cache; q and k, read in whole lines, are loaded nontemporally (not v,
// whose lines two instructions share).  B4 H16 N4096 d128: 234 -> 230 us.
// kOne (walk only): no segment has more than one tile, so nothing is done for a next one.  One tile, B4 H32 N32 d128: 11.1 us
// without it, 10.1 with it.
template <bool kOut, bool kStream, bool kOne>
__global__ __launch_bounds__(f32s::threads(kOut), 2) void fwd_f32_split_kernel(FwdParams p) {
    using namespace f32s;
    constexpr int CT = D / 32;                 // column tiles
    constexpr int KS = parts(kOut);         // waves of a column tile: parts of the key dimension
    constexpr int NW = CT * KS;                // waves
    constexpr int NT = NW * 64;                // threads
    constexpr int DT = D / 32 / KS;            // 32-row tiles of the state that a wave holds
    using Sm = Smem<kOut>;
    constexpr int RS = Sm::RS, RP = Sm::RP, RO = Sm::RO;
    constexpr int PR = D / 4;                  // 16-byte pieces per row
    constexpr int NLOAD = kTile * PR / NT;     // pieces per thread of q and of k
    constexpr int RPP = NT / PR;               // rows one pass of all threads covers
    __shared__ __attribute__((aligned(16))) Sm sm;

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = tid & 63, ln = l & 31, g = l >> 5, l16 = l & 15, q4 = l >> 4;
    const int half = (l >> 4) & 1;
    const int wc = w % CT, wk = KS == 1 ? 0 : w / CT;  // column tile, part of the key dimension
    const int nseg_launch = kOut ? p.nseg : p.nseg - 1;
    const int bh = blockIdx.x / nseg_launch;
    const int seg = blockIdx.x % nseg_launch;
    const int h = bh % p.H;

    const int tok_begin = seg * p.seg_chunks * kChunk;
    const int tok_end = (seg == p.nseg - 1) ? p.N : tok_begin + p.seg_chunks * kChunk;
    const int ntiles = (tok_end - tok_begin + kTile - 1) / kTile;

    const size_t seq_off = (size_t)bh * p.N * D;
    const float* qb = reinterpret_cast<const float*>(p.q) + seq_off;
    const float* kb = reinterpret_cast<const float*>(p.k) + seq_off;
    const float* vb = reinterpret_cast<const float*>(p.v) + seq_off;
    float* ob = static_cast<float*>(p.out) + seq_off;

    // ---- global memory.  Every tile is addressed through buffer descriptors of its L D floats: what lies
    // beyond a ragged tile reads as zero and is not written, with no branch and no clamped address.
    // q, k: piece r of this thread is row RPP r + tid/PR, floats 4(tid%PR)..+3; v: this lane's column, the
    // sixteen keys of its slots; out: row 8m + l/8, floats 32w + 4(l%8)..+3.
    const int j0 = tid / PR, cc = tid % PR;
    const int c_own = 32 * wc + ln;
    f32x4 rq[NLOAD], rk[NLOAD];
    float va[16];  // va[8f + e] = V[key_of(f, e)][c_own]; f = 0: the half of the keys that this wave takes in G2
    auto key_of = [&](int f, int e) { return 16 * (f ^ wk) + 2 * g + (e >> 2) + 4 * (e & 3); };
    const int qk_off = (j0 * D + cc * 4) * 4, v_off = (2 * g * D + c_own) * 4, o_off = ((16 * wk + (l >> 3)) * D + 32 * wc + 4 * (l & 7)) * 4;
    // In the walk a descriptor for each group of rows: what an instruction's immediate offset does not reach would sit in vector
    // registers.  The pre-pass has these, and forming eight descriptors one after the other holds up its loads: with one a
    // tensor, and its one part of a wave known at compile time, B1 H32 N200 26.8 -> 26.4 us, B4 H32 N128 27.1 -> 26.7,
    // B1 H2 N20000 84.9 -> 84.2.
    auto load_qk = [&](int tok0) {
        const auto kt = tile_rsrc(kb, tok0, tok_end);
#pragma unroll
        for (int r = 0; r < NLOAD; ++r) {
            if (kOut) {
                rk[r] = load4<kStream>(tile_rsrc(kb, tok0 + RPP * r, tok_end), qk_off);
                rq[r] = load4<kStream>(tile_rsrc(qb, tok0 + RPP * r, tok_end), qk_off);
            } else {
                rk[r] = load4<kStream>(kt, qk_off + RPP * r * D * 4);
            }
        }
    };
    auto load_v = [&](int tok0, bool both) {
        if (!kOut) {
            const auto vt = tile_rsrc(vb, tok0, tok_end);
#pragma unroll
            for (int x = 0; x < 16; ++x) va[x] = load1(vt, v_off + (16 * (x >> 3) + ((x >> 2) & 1) + 4 * (x & 3)) * D * 4);
            return;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i >= 2 && !both) break;
            const auto vt = tile_rsrc(vb, tok0 + 16 * ((i >> 1) ^ wk) + 8 * (i & 1), tok_end);
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                const int e = 4 * (x >> 1) + 2 * (i & 1) + (x & 1);  // key_of(i >> 1, e)
                va[8 * (i >> 1) + e] = load1(vt, v_off + ((x >> 1) + 4 * (x & 1)) * D * 4);
            }
        }
    };
    load_qk(tok_begin);
    load_v(tok_begin, !kOut);

    {
        const double gd = p.no_decay ? 1.0 : (double)p.gamma[h];
        if (tid < 2) sm.bad[tid] = 0;
        for (int n = tid; n <= kTile; n += NT) {
            const float x = (float)pow_int(gd, n);
            sm.pw[n] = x;
            if (n > 0) sm.lw[n - 1] = x;
            if (n < kTile) {
                auto slot = [](int j) { return (j & 16) + 4 * (j & 3) + ((j >> 2) & 3); };
                const int last = tok_end - tok_begin - (ntiles - 1) * kTile - 1;  // last token of the last tile
                sm.gw[0][slot(kTile - 1 - n)] = x;
                if (n <= last) sm.gw[1][slot(last - n)] = x;
                else sm.gw[1][slot(n)] = 0.0f;  // no token
            }
        }
    }

    // state slice: S[t][r] = S[dk = 32t + pi(m(r, g))][c_own]
    f32x16 S[DT];
    bool bad = false;   // this lane has seen an operand below its least magnitude
    float fin = 0.0f;   // sum of the magnitudes of results: not finite once one of them is not
    auto dk_of = [&](int t, int r) {
        // m = 8(r/4) + 4g + r%4 ; pi swaps the 4- and 8-bits: dk = 16(r/8) + 8g + 4((r/4)&1) + r%4
        return 32 * (DT * wk + t) + 16 * (r >> 3) + 8 * g + 4 * ((r >> 2) & 1) + (r & 3);
    };
    auto load_state = [&](const float* src, f32x16 (&x)[DT]) {
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) x[t][r] = src[dk_of(t, r) * D + c_own];
    };
    auto store_state = [&](float* dst) {
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) dst[dk_of(t, r) * D + c_own] = S[t][r];
    };
    auto enter_state = [&]() {
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) S[t][r] = 0.0f;
        if (kOut) {
            const float* slots = p.seg_state + (size_t)bh * p.state_slots * D * D;
            if (seg == 0) {
                if (p.state_in) load_state(p.state_in + (size_t)bh * D * D, S);
            } else if (!p.fold) {
                load_state(slots + (size_t)(seg * p.state_step - 1) * D * D, S);
            } else {
                // No scan kernel has run: the slots hold the end state T_j of every segment (the first run from
                // the caller's state, the others from zero), and S_in(s) = sum_{j < s} gamma^(L (s-1-j)) T_j.
                const float gl = p.no_decay ? 1.0f : (float)pow_int((double)p.gamma[h], p.seg_chunks * kChunk);
                load_state(slots, S);
#pragma unroll 1
                for (int j = 1; j < seg; ++j) {
                    f32x16 a[DT];
                    load_state(slots + (size_t)j * D * D, a);
#pragma unroll
                    for (int t = 0; t < DT; ++t)
#pragma unroll
                        for (int r = 0; r < 16; ++r) S[t][r] = gl * S[t][r] + a[t][r];
                }
            }
        } else if (p.fold && seg == 0 && p.state_in) {
            load_state(p.state_in + (size_t)bh * D * D, S);
            store_state(p.state_copy + (size_t)bh * D * D);
        }
    };
    enter_state();

    // No wave forms the scores of rows 0..15 with keys 16..31: zero, once.
    if (kOut && !kOne) {
#pragma unroll
        for (int i = 0; i < 2 * CT * kTile * RO / (4 * NT); ++i) reinterpret_cast<f32x4*>(sm.o)[tid + i * NT] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (kOut && tid < 3 * 16 * 2)
        *reinterpret_cast<u32x4*>(&sm.p[(tid >> 5) * kTile * RP + ((tid >> 1) & 15) * RP + 16 + 8 * (tid & 1)]) = u32x4{0, 0, 0, 0};

    __syncthreads();  // tables visible

    // decay weights of the score tile this wave produces (waves 0, 1, 2: (it, jt) = (0,0), (1,0), (1,1));
    // register r of a lane is query 16 it + l16, key 16 jt + q4 + 4 r
    f32x4 wgt;
    if (kOut) {
#pragma unroll
        for (int n = 0; n < 3; ++n) {
            if (n != w) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int d = (n == 1 ? 16 : 0) + l16 - (q4 + 4 * r);  // i - j
                wgt[r] = d >= 0 ? sm.pw[max(d, 0)] : 0.0f;
            }
        }
    }

    // per-lane LDS offsets (elements)
    const int st_off = j0 * RS + cc * 4;                       // staging: + RPP r RS
    const int q_row32 = ln * RS + 32 * DT * wk + 8 * g;                       // G3: + 32 t + 16 h
    const int q_row16 = l16 * RS + 8 * q4;                     // G1: + 16 it RS + 32 s
    const int k_row16 = ((l16 >> 2) + 4 * (l16 & 3)) * RS + 8 * q4;  // G1: + 16 jt RS + 32 s
    const int k_tr0 = (2 * g + 4 * (l16 >> 2)) * RS + 32 * DT * wk + 16 * half + 8 * (l16 & 1) + 4 * ((l16 >> 1) & 1);  // G4: + 32 t, + RS
    const int k_tr[2] = {k_tr0 + 16 * wk * RS, k_tr0 + 16 * (1 ^ wk) * RS};

    // The finished tile of tokens tok0 ..: the two waves of a column tile hold half of the sum each; each adds
    // and stores half of the rows, in whole 128-byte row pieces, all LDS reads before the first store.
    // In the first tile of the walk there is none: what is read is zero, and `on` = 0 stores nothing.
    struct OutHalves {
        f32x4 x[2][2];
    };
    auto read_out = [&]() {
        OutHalves v;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const float* src = sm.o + wc * (kTile * RO) + (16 * wk + 8 * m + (l >> 3)) * RO + 4 * (l & 7);
            v.x[m][0] = *reinterpret_cast<const f32x4*>(src);
            v.x[m][1] = *reinterpret_cast<const f32x4*>(src + CT * kTile * RO);
        }
        return v;
    };
    auto store_out = [&](const OutHalves& v, int tok0, bool on) {
        const auto ot = tile_rsrc(ob, tok0, on ? tok_end : tok0);
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const f32x4 val = v.x[m][0] + v.x[m][1];
#pragma unroll
            for (int x = 0; x < 4; ++x) fin += __builtin_fabsf(val[x]);
            store4_nt(val, ot, o_off + 8 * m * D * 4);
        }
    };

    // Least magnitudes of operands other than zero: two that are multiplied make 2^-96 or more, of which the terms and
    // partial sums that the matrix instructions drop (below 2^-126) are less than a rounding, and none is below 2^-100,
    // where its own last terms would go.  `tilt` shares the range out by the scales of a segment's first token, q's against
    // k's, in the pre-pass v's against k's: it decides what is out of range, never what is right.
    const float far = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(sm.pw[kTile - 1])));  // gamma^31
    const int scale = exponent4((kOut ? qb : vb) + (size_t)tok_begin * D) - exponent4(kb + (size_t)tok_begin * D);
    const int tilt = __builtin_amdgcn_readfirstlane(min(max(scale / 2, -48), 48));
    const float least_q = pow2(-52 + tilt), least_k = pow2(-44 - tilt);  // S: as k
    const float least_p = pow2(-52 - tilt);
    // Gam V, whose least is q's, is gamma^31 V or more (or zero, with gamma = 0)
    const float least_v = far > 0.0f ? fmaxf(pow2(-44 + tilt), pow2(-52 + tilt) / far) : pow2(-44 + tilt);

    // The walk with split products.  True: an operand or a result was out of range somewhere, and nothing of what
    // the walk has made stands.
    auto walk_split = [&]() -> bool {
        auto k_at = [&](int x) { return rk[x >> 2][x & 3]; };
        auto q_at = [&](int x) { return rq[x >> 2][x & 3]; };
        auto s_at = [&](int x) { return S[x >> 4][x & 15]; };
        uint32_t s_small = ~0u;
        // The operands of the tile to come: k, q and, an operand in G3 only, S.  In the walk without a branch but for S: one costs
        // as much as some twenty vector operations, and between MFMAs these cost little.
        auto watch_qk = [&]() {
            if (kOut) bad |= (smallest_nonzero<4 * NLOAD>(k_at) < rank_nonzero(least_k)) | (smallest_nonzero<4 * NLOAD>(q_at) < rank_nonzero(least_q));
            else bad |= has_small<4 * NLOAD>(k_at, least_k);
        };
        auto watch_s = [&]() {
            s_small = ~0u;
            if (__any(smallest<16 * DT>(s_at) < least_k)) s_small = smallest_nonzero<16 * DT>(s_at);
        };
        // piece r of k and q as planes, to buffer b
        auto stage = [&](int b, int r) {
            store4(sm.k[b] + st_off + RPP * r * RS, kTile * RS, rk[r][0], rk[r][1], rk[r][2], rk[r][3]);
            if (kOut) store4(sm.q + st_off + RPP * r * RS, kTile * RS, rq[r][0], rq[r][1], rq[r][2], rq[r][3]);
        };
        // (a tile beyond the last reads as zero, without an access to memory)
        auto tile_at = [&](int t) { return tok_begin + t * kTile; };

        // the entering state arrives here, not at its first use in the loop: there every tile would wait for all loads
#pragma unroll
        for (int t = 0; t < DT; ++t) asm("" : "+v"(S[t]));
        // The walk splits a tile's k and q while it works on the tile before; the pre-pass, where two workgroups share a
        // compute unit and one splits while the other multiplies, has no registers left for that.
        auto stage_tile = [&](int t) {
            watch_qk();
#pragma unroll
            for (int r = 0; r < NLOAD; ++r) stage(t & 1, r);
        };
        if (kOut) {
            watch_s();
            stage_tile(0);
            if (!kOne) load_qk(tile_at(1));
        }
        int stop = 0;
        for (int t = 0; t < (kOne ? 1 : ntiles); ++t) {
            const int tok0 = tok_begin + t * kTile;
            const int Lc = min(kTile, tok_end - tok0);
            uint16_t* kt = sm.k[t & 1];

            if (!kOut) stage_tile(t);
            __syncthreads();  // this tile's planes and the previous one's sums visible; everyone is done reading its planes and scores
            // Something out of range up to the tile before?  Written in even tiles and read in odd ones: not both between two
            // barriers, or the waves could disagree.  us, all in range / all out of range, B9 H33 N2000, B16 H32 N300: every tile
            // 554 / 834, 121 / 161; every second 542 / 825, 117 / 151; every eighth 541 / 882, 117 / 218.
            if (t % 2 == 1 && __builtin_amdgcn_readfirstlane(sm.bad[0])) {
                stop = 1;
                break;
            }
            if (!kOut) load_qk(tile_at(t + 1));
            // A state that has decayed below its least magnitude is held against the rows of q that it meets: with
            // tokens of zeros behind a sequence there are none.
            if (kOut && __any(s_small < rank_nonzero(least_k))) {
                uint32_t q_small = ~0u;
#pragma unroll
                for (int i = 0; i < 2 * DT; ++i) {
                    const u32x4 x = *reinterpret_cast<const u32x4*>(&sm.q[q_row32 + 16 * i]);  // upper halves
#pragma unroll
                    for (int e = 0; e < 4; ++e) q_small = min(q_small, min((x[e] << 17) - 1, ((x[e] & 0xffff0000u) << 1) - 1));
                }
#pragma unroll
                for (int m = 1; m < 64; m *= 2) q_small = min(q_small, (uint32_t)__shfl_xor((int)q_small, m));
                const float sv = __uint_as_float((s_small + 1) >> 1), qv = __uint_as_float((q_small + 1) >> 1);
                bad |= s_small != ~0u && q_small != ~0u && (sv < 0x1p-100f || sv * qv < 0x1p-96f);
            }

            auto v_at = [&](int x) { return va[x]; };
            bad |= kOut ? smallest_nonzero<8>(v_at) < rank_nonzero(least_v) : has_small<16>(v_at, least_v);
            if (t % 2 == 0 && __any(bad | !(fin < __builtin_inff()))) sm.bad[0] = 1;
            // Gam V as operands, half f of the slots
            Frag3 gv[2];
            const float* gw = sm.gw[t == ntiles - 1];
            f32x4 wv[2];
            auto read_weights = [&](int f) {
#pragma unroll
                for (int u = 0; u < 2; ++u) wv[u] = *reinterpret_cast<const f32x4*>(&gw[16 * (f ^ wk) + 8 * g + 4 * u]);
            };
            auto weigh = [&](int f) {
#pragma unroll
                for (int e = 0; e < 8; ++e) wv[e >> 2][e & 3] *= va[8 * f + e];
#pragma unroll
                for (int e = 0; e < 4; ++e) put2(gv[f], e, wv[e >> 1][2 * (e & 1)], wv[e >> 1][2 * (e & 1) + 1]);
            };
            f32x16 o, os;  // leading products, the others
            Frag3 vo, po;  // G2: V, the half of the keys that this wave takes; the scores
            if (kOut) {
                // G1 + mask for the score tile this wave produces
#pragma unroll
                for (int n = 0; n < 3; ++n) {
                    if (n != w) continue;
                    const int it = n > 0, jt = n > 1;
                    f32x4 big = {0.f, 0.f, 0.f, 0.f}, small = {0.f, 0.f, 0.f, 0.f};
                    auto read = [&](Frag3& a, Frag3& b, int s) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            a.x[i] = *reinterpret_cast<const u32x4*>(&kt[i * kTile * RS + k_row16 + 16 * jt * RS + 32 * s]);
                            b.x[i] = *reinterpret_cast<const u32x4*>(&sm.q[i * kTile * RS + q_row16 + 16 * it * RS + 32 * s]);
                        }
                    };
                    Frag3 a[3], b[3];
                    read(a[0], b[0], 0);
                    read(a[1], b[1], 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int s = 0; s < D / 32; ++s) {
                        if (s + 2 < D / 32) read(a[(s + 2) % 3], b[(s + 2) % 3], s + 2);
                        small = mma16_small(a[s % 3], b[s % 3], small);
                        big = mfma16(a[s % 3].x[0], b[s % 3].x[0], big);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    float m[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool below = n == 1 || l16 >= q4 + 4 * r;  // on or below the diagonal
                        m[r] = below ? (big[r] + small[r]) * wgt[r] : 0.0f;
                    }
                    bad |= smallest_nonzero<4>([&](int x) { return m[x]; }) < rank_nonzero(least_p);
                    store4(sm.p + (16 * it + l16) * RP + 16 * jt + 4 * q4, kTile * RP, m[0], m[1], m[2], m[3]);
                }

                __builtin_amdgcn_sched_barrier(0);
                // G3: O = Q S, rows of O scaled by gamma^(i+1).  The operands of step s + 1 are read and split
                // between the MFMAs of step s.
#pragma unroll
                for (int r = 0; r < 16; ++r) o[r] = os[r] = 0.0f;
                auto read = [&](Frag3& a, Frag3& b, int s) {
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        a.x[i] = *reinterpret_cast<const u32x4*>(&sm.q[i * kTile * RS + q_row32 + 16 * s]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) put2(b, e, S[s >> 1][8 * (s & 1) + 2 * e], S[s >> 1][8 * (s & 1) + 2 * e + 1]);
                };
                Frag3 a[2], b[2];
                const OutHalves done = read_out();
                read(a[0], b[0], 0);
                if (!kOne) store_out(done, tok0 - kTile, t > 0);
                __builtin_amdgcn_sched_barrier(0);
                f32x4 lam[4];
#pragma unroll
                for (int s = 0; s < 2 * DT; ++s) {
                    if (s + 1 < 2 * DT) read(a[(s + 1) & 1], b[(s + 1) & 1], s + 1);
                    if (s == 2 * DT - 3) read_weights(0);
                    if (s == 2 * DT - 2) weigh(0);
                    if (s == 2 * DT - 1) {
#pragma unroll
                        for (int i = 0; i < 3; ++i) sm.gv[w][i][l] = gv[0].x[i];
#pragma unroll
                        for (int u = 0; u < 4; ++u) lam[u] = *reinterpret_cast<const f32x4*>(&sm.lw[8 * u + 4 * g]);
                    }
                    os = mma32_small(a[s & 1], b[s & 1], os);
                    o = ElemBf16::mfma32(a[s & 1].x[0], b[s & 1].x[0], o);
                    // LDS reads, then MFMAs and vector operations in turn
                    if (s + 1 < 2 * DT) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
                    if (s == 2 * DT - 2) interleave<8, 12>();
                    else interleave<8, 6>();
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) o[r] = __builtin_fmaf(os[r], lam[r >> 2][r & 3], o[r] * lam[r >> 2][r & 3]);
            } else {
                read_weights(0);
                weigh(0);
                read_weights(1);
                weigh(1);
                __builtin_amdgcn_sched_barrier(0);
                load_v(tile_at(t + 1), true);
                __builtin_amdgcn_sched_barrier(0);
            }
            // G4: S = gamma^L S + K^T (Gam V), one 32-row tile after the other
            auto read_k = [&](Frag3& a, int dt, int f) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const uint16_t* src = &kt[i * kTile * RS + k_tr[f] + 32 * dt];
                    const u32x2 lo = lds_tr(src), hi = lds_tr(src + RS);
                    a.x[i] = u32x4{lo.x, lo.y, hi.x, hi.y};
                }
            };
            const float gl = sm.pw[Lc];
            Frag3 a[4];
            read_k(a[0], 0, 0);
            if (kOut) {
                __syncthreads();  // scores and weighted values visible
#pragma unroll
                for (int i = 0; i < 3; ++i) gv[1].x[i] = sm.gv[w ^ CT][i][l];
            }
            read_k(a[1], 0, 1);
            __builtin_amdgcn_sched_barrier(0);
            f32x16 sb[2], ss[2], pb, ps;  // leading products, the others
            auto add_up = [&](int dt) {
#pragma unroll
                for (int r = 0; r < 16; ++r) S[dt][r] = __builtin_fmaf(S[dt][r], gl, sb[dt & 1][r] + ss[dt & 1][r]);
            };
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const int n = dt & 1, c = 2 * n;
                if (!kOut && dt + 1 < DT) {
                    read_k(a[c ^ 2], dt + 1, 0);
                    read_k(a[(c ^ 2) + 1], dt + 1, 1);
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) sb[n][r] = ss[n][r] = 0.0f;
                ss[n] = mma32_small(a[c], gv[0], ss[n]);
                sb[n] = ElemBf16::mfma32(a[c].x[0], gv[0].x[0], sb[n]);
                ss[n] = mma32_small(a[c + 1], gv[1], ss[n]);
                sb[n] = ElemBf16::mfma32(a[c + 1].x[0], gv[1].x[0], sb[n]);
                auto stage_next = [&](int r) {
                    if (!kOne) stage((t + 1) & 1, r);
                };
                if (kOut && dt == 0) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) put2(vo, e, va[2 * e], va[2 * e + 1]);
                    stage_next(0);
                    if (!kOne) watch_qk();
#pragma unroll
                    for (int i = 0; i < 3; ++i) po.x[i] = *reinterpret_cast<const u32x4*>(&sm.p[i * kTile * RP + ln * RP + 16 * wk + 8 * g]);
                }
                if (kOut && dt == 1) {
                    stage_next(1);
                    float* mine = sm.o + w * (kTile * RO);
#pragma unroll
                    for (int r = 0; r < 16; ++r) mine[(8 * (r >> 2) + 4 * g + (r & 3)) * RO + ln] = o[r] + (pb[r] + ps[r]);
                }
                if (kOut) interleave<16, 6>();
                if (!kOut || dt > 0) add_up(dt);
                __builtin_amdgcn_sched_barrier(0);
                if (kOut && dt == 0) {
                    if (!kOne) load_v(tile_at(t + 1), false);
                    __builtin_amdgcn_sched_barrier(0);
                    // G2: P V, over one half of the keys.  Both waves leave their sums for store_out.  P V has accumulators of its
                    // own: in those of G3 the matrix instructions would take a far decayed Lam (Q S) as zero.
#pragma unroll
                    for (int r = 0; r < 16; ++r) pb[r] = ps[r] = 0.0f;
                    read_k(a[2], 1, 0);
                    read_k(a[3], 1, 1);
                    ps = mma32_small(po, vo, ps);
                    pb = ElemBf16::mfma32(po.x[0], vo.x[0], pb);
                    add_up(0);
                    interleave<8, 6>();
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (kOut && !kOne) {
                watch_s();
                load_qk(tile_at(t + 2));
            }
        }

        if (kOut) {
            __syncthreads();  // the last tile's sums visible
            store_out(read_out(), tok_begin + (ntiles - 1) * kTile, !stop);
        }
#pragma unroll
        for (int x = 0; x < 16 * DT; ++x) fin += __builtin_fabsf(S[x >> 4][x & 15]);  // not finite once, not finite for good
        if (__any(bad | !(fin < __builtin_inff()))) sm.bad[1] = 1;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(sm.bad[1]) != 0;
    };

    // The same walk with fp32 matrix instructions on fp32 tiles in the same LDS: same waves, same column tiles and
    // accumulators, same slots.  Right for every operand; B4 H16 N4096 308 us a call.
    auto walk_fp32 = [&]() {
        constexpr int RF = D + 4, RPF = kTile + 4;  // row strides (floats)
        float* kf = reinterpret_cast<float*>(&sm.k[0][0]);
        float* qf = reinterpret_cast<float*>(&sm.q[0]);
        float* pf = reinterpret_cast<float*>(&sm.p[0]);
        const int k_row = (l16 >> 2) + 4 * (l16 & 3);                  // G1: key of accumulator row l16, + 16 jt
        const int pi = (ln & 19) | ((ln & 4) << 1) | ((ln & 8) >> 1);  // G4: key index of accumulator row ln
        for (int t = 0; t < ntiles; ++t) {
            const int tok0 = tok_begin + t * kTile;
            const int next = tok_begin + min(t + 1, ntiles - 1) * kTile;
            const int Lc = min(kTile, tok_end - tok0);
            if (t > 0) {
                __syncthreads();
                if (kOut) store_out(read_out(), tok0 - kTile, true);
            }
#pragma unroll
            for (int r = 0; r < NLOAD; ++r) {
                *reinterpret_cast<f32x4*>(kf + (j0 + RPP * r) * RF + 4 * cc) = rk[r];
                if (kOut) *reinterpret_cast<f32x4*>(qf + (j0 + RPP * r) * RF + 4 * cc) = rq[r];
            }
            __syncthreads();
            load_qk(next);
            if (kOut) {
#pragma unroll
                for (int n = 0; n < 3; ++n) {  // G1
                    if (n != w) continue;
                    const int it = n > 0, jt = n > 1;
                    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
                    for (int s = 0; s < D / 16; ++s) {
                        const f32x4 a = *reinterpret_cast<const f32x4*>(kf + (16 * jt + k_row) * RF + 16 * s + 4 * q4);
                        const f32x4 b = *reinterpret_cast<const f32x4*>(qf + (16 * it + l16) * RF + 16 * s + 4 * q4);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0);
                    }
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool below = n == 1 || l16 >= q4 + 4 * r;
                        acc[r] = below ? acc[r] * wgt[r] : 0.0f;
                    }
                    *reinterpret_cast<f32x4*>(pf + (16 * it + l16) * RPF + 16 * jt + 4 * q4) = acc;
                }
                f32x16 o;  // G3
#pragma unroll
                for (int r = 0; r < 16; ++r) o[r] = 0.0f;
#pragma unroll
                for (int x = 0; x < 4 * DT; ++x) {
                    const f32x4 a = *reinterpret_cast<const f32x4*>(qf + ln * RF + dk_of(x >> 2, 4 * (x & 3)));
#pragma unroll
                    for (int e = 0; e < 4; ++e) o = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e], S[x >> 2][4 * (x & 3) + e], o, 0, 0, 0);
                }
                float* mine = sm.o + w * (kTile * RO);
                auto put_rows = [&](int r0, int r1) {
#pragma unroll
                    for (int r = r0; r < r1; ++r) mine[(8 * (r >> 2) + 4 * g + (r & 3)) * RO + ln] = o[r];
                };
#pragma unroll
                for (int r = 0; r < 16; ++r) o[r] *= sm.lw[8 * (r >> 2) + 4 * g + (r & 3)];
                __syncthreads();  // scores visible
#pragma unroll
                for (int f = 0; f < 2; ++f) {  // G2, as above: keys 16..31 do not reach rows 0..15
                    if (f != wk) continue;
                    if (f == 1) put_rows(0, 8);
                    const float* row = pf + ln * RPF + 16 * f + 8 * g;
                    const f32x4 a[2] = {*reinterpret_cast<const f32x4*>(row), *reinterpret_cast<const f32x4*>(row + 4)};
#pragma unroll
                    for (int e = 0; e < 8; ++e) o = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e >> 2][e & 3], va[e], o, 0, 0, 0);
                    put_rows(f == 1 ? 8 : 0, 16);
                }
            }
            float gva[16];
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const int back = Lc - 1 - key_of(x >> 3, x & 7);
                gva[x] = back >= 0 ? va[x] * sm.pw[max(back, 0)] : 0.0f;
            }
            load_v(next, true);
            const float gl = sm.pw[Lc];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {  // G4
                S[dt] *= gl;
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    const float a = kf[key_of(x >> 3, x & 7) * RF + 32 * (DT * wk + dt) + pi];
                    S[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, gva[x], S[dt], 0, 0, 0);
                }
            }
        }
        if (kOut) {
            __syncthreads();
            store_out(read_out(), tok_begin + (ntiles - 1) * kTile, true);
        }
    };

    // A decay this fast takes scores and values out of range as a rule; otherwise the split walk finds out.
    bool fp32 = far < 0x1p-20f && __builtin_amdgcn_readfirstlane(sm.pw[1] > 0.0f);
    if (!fp32 && walk_split()) {
        load_qk(tok_begin);
        enter_state();
        fp32 = true;
    }
    if (fp32) {
        load_v(tok_begin, true);
        walk_fp32();
    }

    float* dst = nullptr;
    if (kOut) {
        if (seg == p.nseg - 1 && p.state_out) dst = p.state_out + (size_t)bh * D * D;
    } else {
        dst = p.seg_state + ((size_t)bh * p.state_slots + seg) * D * D;
    }
    if (dst) store_state(dst);
}

namespace {
template <bool kOut>
hipError_t launch(const FwdParams& p, int blocks, hipStream_t stream) {
    const dim3 grid(blocks), block(f32s::threads(kOut));
    if (kOut && p.nseg == 1 && p.N <= f32s::kTile) hipLaunchKernelGGL((fwd_f32_split_kernel<kOut, false, kOut>), grid, block, 0, stream, p);
    else if (p.stream_loads) hipLaunchKernelGGL((fwd_f32_split_kernel<kOut, true, false>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((fwd_f32_split_kernel<kOut, false, false>), grid, block, 0, stream, p);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_fwd_f32_split_states(const FwdParams& p, int BH, hipStream_t stream) {
    return p.nseg <= 1 ? hipSuccess : launch<false>(p, BH * (p.nseg - 1), stream);
}

hipError_t launch_fwd_f32_split_walk(const FwdParams& p, int BH, hipStream_t stream) {
    return launch<true>(p, BH * p.nseg, stream);
}

}  // namespace leet
