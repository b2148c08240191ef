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
// results stand for every operand.  Ordinary data never does that (nor zeros behind a sequence: B4 H16 N4096, half of it
// zeros, 252 us); the watching costs some 50 of 650 vector operations
// a tile (B4 H16 N4096 273 -> 282 us; without it q, k ~ 2^-60 with v ~ 2^104 came out with errors of 6e-4).
//
// Work split: a column tile of 32 value columns belongs to two waves (in the pre-pass: one),
// which hold half of the key dimension each: S[half of dk][cols] in fp32 accumulators for the whole walk.
// Each computes its half of the sum Q S and the scores' product with one half of the keys; the two sums
// meet in LDS on their way out.  Eight waves, one workgroup a compute unit; in the pre-pass four and two.
//
// What bounds it: matrix and vector instructions, which take turns on a SIMD more than they overlap: per
// 32-token tile 624 MFMAs of 32 cycles (of 4 SIMDs) and, per wave, some 650 vector operations, most of them
// splits.  Against a kernel on fp32 MFMAs, one device: B4 H16 N4096 319 -> 282 us, B1 H32 N777 53.5 -> 45.9, B1 H300 N2000
// 819 -> 630 (walk_fp32 alone, B1 H300 N2000: 805).
// Against 64 bits a single product errs by at most 5.99e-8 of itself (5.95e-8 with fp32 MFMAs).  Sums round less
// often: over forty sizes outputs 0.66e-7..0.95e-7 in the 2-norm (1.5e-7..2.8e-7), states 0.33 to 0.83 of what fp32
// MFMAs give; the largest single error of a state after two tokens, in units of its rms and over 200 seeds, is 4.2e-7 on
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

// The pre-pass (kOut = false) reads no Q and forms no scores; it has two K buffers instead and so
// one barrier a tile.
template <bool kOut>
struct Smem {
    static constexpr int RS = D + 8;    // padded row strides (elements)
    static constexpr int RP = kTile + 8;
    static constexpr int RO = kTile + 8;  // output scratch of a wave (floats)
    uint16_t k[kOut ? 1 : 2][3 * kTile * RS];   // three planes each
    uint16_t q[kOut ? 3 * kTile * RS : 8];
    uint16_t p[kOut ? 3 * kTile * RP : 8];      // masked scores P[i][slot]
    float o[kOut ? 2 * (D / 32) * kTile * RO : 4];  // output tiles of the waves
    float lw[kTile];       // gamma^(i+1)
    float gw[kTile];       // gamma^(31-j) in slot order
    float pw[kTile + 4];   // gamma^n, n = 0..32
    int bad[3];            // out of range: seen in even tiles, in odd tiles, in the whole walk
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

// The tile of tokens tok0 .. min(tok0 + 31, tok_end - 1) of a tensor with rows of D floats.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const float* base, int tok0, int tok_end) {
    // all of it is the same in every lane; the compiler is told, since it moves part of the arithmetic to vector registers
    const uintptr_t addr = reinterpret_cast<uintptr_t>(base) + (size_t)tok0 * (D * 4);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)addr), hi = __builtin_amdgcn_readfirstlane((uint32_t)(addr >> 32));
    const int bytes = __builtin_amdgcn_readfirstlane(min(kTile, tok_end - tok0) * (D * 4));
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
template <bool kOut, bool kStream>
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
    const int wc = w % CT, wk = w / CT;  // column tile, part of the key dimension
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
    float va[16];  // va[8f + e] = V[key_of(f, e)][c_own]
    auto key_of = [&](int f, int e) { return 16 * f + 2 * g + (e >> 2) + 4 * (e & 3); };
    const int qk_off = (j0 * D + cc * 4) * 4, v_off = (2 * g * D + c_own) * 4, o_off = ((16 * wk + (l >> 3)) * D + 32 * wc + 4 * (l & 7)) * 4;
    auto load_qk = [&](int tok0) {
        const auto kt = tile_rsrc(kb, tok0, tok_end);
        const auto qt = tile_rsrc(qb, tok0, tok_end);
#pragma unroll
        for (int r = 0; r < NLOAD; ++r) {
            rk[r] = load4<kStream>(kt, qk_off + RPP * r * D * 4);
            if (kOut) rq[r] = load4<kStream>(qt, qk_off + RPP * r * D * 4);
        }
    };
    auto load_v = [&](int tok0) {
        const auto vt = tile_rsrc(vb, tok0, tok_end);
#pragma unroll
        for (int x = 0; x < 16; ++x) va[x] = load1(vt, v_off + (16 * (x >> 3) + ((x >> 2) & 1) + 4 * (x & 3)) * D * 4);
    };
    load_qk(tok_begin);
    load_v(tok_begin);

    {
        const double gd = p.no_decay ? 1.0 : (double)p.gamma[h];
        if (tid < 3) sm.bad[tid] = 0;
        for (int n = tid; n <= kTile; n += NT) {
            const float x = (float)pow_int(gd, n);
            sm.pw[n] = x;
            if (n > 0) sm.lw[n - 1] = x;
            if (n < kTile) {
                const int j = kTile - 1 - n;  // slot 16(j/16) + 4(j%4) + (j/4)%4
                sm.gw[(j & 16) + 4 * (j & 3) + ((j >> 2) & 3)] = x;
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
    const int k_tr = (2 * g + 4 * (l16 >> 2)) * RS + 32 * DT * wk + 16 * half + 8 * (l16 & 1) + 4 * ((l16 >> 1) & 1);  // G4: + 16 f RS + 32 t, + RS

    // The finished tile of tokens tok0 ..: the two waves of a column tile hold half of the sum each; each adds
    // and stores half of the rows, in whole 128-byte row pieces, all LDS reads before the first store.
    auto store_out = [&](int tok0) {
        f32x4 val[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const float* src = sm.o + wc * (kTile * RO) + (16 * wk + 8 * m + (l >> 3)) * RO + 4 * (l & 7);
            val[m] = *reinterpret_cast<const f32x4*>(src) + *reinterpret_cast<const f32x4*>(src + CT * kTile * RO);
        }
#pragma unroll
        for (int x = 0; x < 8; ++x) fin += __builtin_fabsf(val[x >> 2][x & 3]);
        const auto ot = tile_rsrc(ob, tok0, tok_end);
#pragma unroll
        for (int m = 0; m < 2; ++m) store4_nt(val[m], ot, o_off + 8 * m * D * 4);
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
        // the entering state arrives here, not at its first use in the loop: there every tile would wait for all loads
#pragma unroll
        for (int t = 0; t < DT; ++t) asm("" : "+v"(S[t]));
        int stop = 0;
        for (int t = 0; t < ntiles; ++t) {
            const int tok0 = tok_begin + t * kTile;
            const int next = tok_begin + min(t + 1, ntiles - 1) * kTile;
            const int Lc = min(kTile, tok_end - tok0);
            uint16_t* kt = sm.k[kOut ? 0 : (t & 1)];

            if (kOut && t > 0) {
                __syncthreads();  // the previous tile's sums visible; everyone is done reading its planes and scores
                store_out(tok0 - kTile);
            }
            auto k_at = [&](int x) { return rk[x / 4][x % 4]; };
            auto s_at = [&](int x) { return S[x / 16][x % 16]; };
            float least_seen = smallest<4 * NLOAD>(k_at);
            if (kOut) least_seen = __builtin_fminf(least_seen, smallest<16 * DT>(s_at));  // S is an operand in G3 only
            uint32_t s_small = ~0u;
            if (__any(least_seen < least_k)) {
                bad |= smallest_nonzero<4 * NLOAD>(k_at) < rank_nonzero(least_k);
                if (kOut) s_small = smallest_nonzero<16 * DT>(s_at);
            }
            if (kOut) bad |= has_small<4 * NLOAD>([&](int x) { return rq[x >> 2][x & 3]; }, least_q);
#pragma unroll
            for (int r = 0; r < NLOAD; ++r) {
                store4(kt + st_off + RPP * r * RS, kTile * RS, rk[r][0], rk[r][1], rk[r][2], rk[r][3]);
                if (kOut) store4(sm.q + st_off + RPP * r * RS, kTile * RS, rq[r][0], rq[r][1], rq[r][2], rq[r][3]);
            }
            __syncthreads();
            // Something out of range in the tile before?  (Its flag is not written again before the next barrier.)
            stop = sm.bad[(t & 1) ^ 1];
            // The next tile's loads, in flight during the MFMA work below; the last tile loads itself again.  (Under
            // a condition, every later wait would have to cover the path without them and so drain them.)
            load_qk(next);
            __builtin_amdgcn_sched_barrier(0);
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

            f32x16 o, os;  // leading products, the others
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
                    Frag3 a[2], b[2];
                    read(a[0], b[0], 0);
#pragma unroll
                    for (int s = 0; s < D / 32; ++s) {
                        if (s + 1 < D / 32) read(a[(s + 1) & 1], b[(s + 1) & 1], s + 1);
                        small = mma16_small(a[s & 1], b[s & 1], small);
                        big = mfma16(a[s & 1].x[0], b[s & 1].x[0], big);
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
                read(a[0], b[0], 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 2 * DT; ++s) {
                    if (s + 1 < 2 * DT) read(a[(s + 1) & 1], b[(s + 1) & 1], s + 1);
                    os = mma32_small(a[s & 1], b[s & 1], os);
                    o = ElemBf16::mfma32(a[s & 1].x[0], b[s & 1].x[0], o);
                    __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);  // LDS reads, then MFMAs and vector operations in turn
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x2, 6, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const f32x4 lam = *reinterpret_cast<const f32x4*>(&sm.lw[8 * u + 4 * g]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[4 * u + r] = __builtin_fmaf(os[4 * u + r], lam[r], o[4 * u + r] * lam[r]);
                }

                __syncthreads();  // scores visible
                // G2: P V.  Wave part 0 takes keys 0..15, part 1 keys 16..31, which do not reach rows 0..15 (registers 0..7);
                // both leave their sums for store_out.  P V has accumulators of its own: in those of G3 the matrix instructions
                // would take a far decayed Lam (Q S) as zero.
                float* mine = sm.o + w * (kTile * RO);
#pragma unroll
                for (int f = 0; f < 2; ++f) {
                    if (f != wk) continue;
                        Frag3 a, b;
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        a.x[i] = *reinterpret_cast<const u32x4*>(&sm.p[i * kTile * RP + ln * RP + 16 * f + 8 * g]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) put2(b, e, va[8 * f + 2 * e], va[8 * f + 2 * e + 1]);
                    f32x16 c, cs;
#pragma unroll
                    for (int r = 0; r < 16; ++r) c[r] = cs[r] = 0.0f;
                    cs = mma32_small(a, b, cs);
                    c = ElemBf16::mfma32(a.x[0], b.x[0], c);
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        mine[(8 * (r >> 2) + 4 * g + (r & 3)) * RO + ln] = f == 1 && r < 8 ? o[r] : o[r] + (c[r] + cs[r]);
                }
            }

            bad |= has_small<16>([&](int x) { return va[x]; }, least_v);
            // Gam V as operands; with them the registers of V are free for the next tile's loads.
            Frag3 gv[2];
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                f32x4 wv[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) wv[u] = *reinterpret_cast<const f32x4*>(&sm.gw[16 * f + 8 * g + 4 * u]);
                if (Lc < kTile) {  // ragged: gamma^(L-1-j)
#pragma unroll
                    for (int e = 0; e < 8; ++e) wv[e >> 2][e & 3] = sm.pw[max(Lc - 1 - key_of(f, e), 0)];
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) wv[e >> 2][e & 3] *= va[8 * f + e];
    #pragma unroll
                for (int e = 0; e < 4; ++e) put2(gv[f], e, wv[e >> 1][2 * (e & 1)], wv[e >> 1][2 * (e & 1) + 1]);
            }
            if (__any(bad | !(fin < __builtin_inff()))) sm.bad[t & 1] = 1;
            __builtin_amdgcn_sched_barrier(0);
            load_v(next);
            __builtin_amdgcn_sched_barrier(0);
            // G4: S = gamma^L S + K^T (Gam V)
            {
                const float gl = sm.pw[Lc];
                auto read = [&](Frag3& a, int u) {  // step u: tile u/2, slots 16 (u%2) ..
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const uint16_t* src = &kt[i * kTile * RS + k_tr + 16 * (u & 1) * RS + 32 * (u >> 1)];
                        const u32x2 lo = lds_tr(src), hi = lds_tr(src + RS);
                        a.x[i] = u32x4{lo.x, lo.y, hi.x, hi.y};
                    }
                };
                Frag3 a[4];
                read(a[0], 0);
                read(a[1], 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const int c = 2 * (dt & 1);
                    if (dt + 1 < DT) {
                        read(a[c ^ 2], 2 * dt + 2);
                        read(a[(c ^ 2) + 1], 2 * dt + 3);
                    }
                    f32x16 sb, ss;  // leading products, the others
#pragma unroll
                    for (int r = 0; r < 16; ++r) sb[r] = ss[r] = 0.0f;
                    ss = mma32_small(a[c], gv[0], ss);
                    ss = mma32_small(a[c + 1], gv[1], ss);
                    sb = ElemBf16::mfma32(a[c].x[0], gv[0].x[0], sb);
                    sb = ElemBf16::mfma32(a[c + 1].x[0], gv[1].x[0], sb);
#pragma unroll
                    for (int r = 0; r < 16; ++r) S[dt][r] = __builtin_fmaf(S[dt][r], gl, sb[r] + ss[r]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (__builtin_amdgcn_readfirstlane(stop)) break;
        }

        if (kOut) {
            __syncthreads();  // the last tile's sums visible
            if (!stop) store_out(tok_begin + (ntiles - 1) * kTile);
        }
#pragma unroll
        for (int x = 0; x < 16 * DT; ++x) fin += __builtin_fabsf(S[x >> 4][x & 15]);  // not finite once, not finite for good
        if (__any(bad | !(fin < __builtin_inff()))) sm.bad[2] = 1;
        __syncthreads();
        return __builtin_amdgcn_readfirstlane(sm.bad[2]) != 0;
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
                if (kOut) store_out(tok0 - kTile);
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
                    for (int e = 0; e < 8; ++e) o = __builtin_amdgcn_mfma_f32_32x32x2f32(a[e >> 2][e & 3], va[8 * f + e], o, 0, 0, 0);
                    put_rows(f == 1 ? 8 : 0, 16);
                }
            }
            float gva[16];
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const int back = Lc - 1 - key_of(x >> 3, x & 7);
                gva[x] = back >= 0 ? va[x] * sm.pw[max(back, 0)] : 0.0f;
            }
            load_v(next);
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
            store_out(tok_begin + (ntiles - 1) * kTile);
        }
    };

    // A decay this fast takes scores and values out of range as a rule; otherwise the split walk finds out.
    bool fp32 = far < 0x1p-20f && __builtin_amdgcn_readfirstlane(sm.pw[1] > 0.0f);
    if (!fp32 && walk_split()) {
        load_qk(tok_begin);
        load_v(tok_begin);
        enter_state();
        fp32 = true;
    }
    if (fp32) walk_fp32();

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
    if (p.stream_loads) hipLaunchKernelGGL((fwd_f32_split_kernel<kOut, true>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((fwd_f32_split_kernel<kOut, false>), grid, block, 0, stream, p);
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
