// Matrix-core kernel (gfx950 / CDNA4).  Described for fp16 coefficients, the
// headline case; fp32 and 8-bit coefficients differ only in stage 3's operand
// handling (end of this comment).
//
// One fused, persistent kernel does stage 1 (up-sampling), stage 3
// (F_i = Phi_i D, paper Eq. 2) and stage 4 (y_i = F_i B_i^T) for tiles of HR
// pixels; neither F nor B of Eq. 3 ever reaches memory.  The only large stream
// is the coefficient tensor Phi (L planes, fp16), read exactly once.
//
// Stage 3 is a (taps x atoms) . (atoms x pixels) product per wavefront:
//
//     A = D^T, rows = filter taps (padded to 32), K = atoms  (constant per launch)
//     B = Phi, K = atoms, columns = 32 pixels                 (streamed from HBM)
//     v_mfma_f32_32x32x16_f16 (+ one v_mfma_f32_32x32x8_f16 when L % 16 == 8)
//
// The dictionary is fp32; it enters as hi + lo fp16 halves (two MFMAs per
// step), so the only rounding left is the one already in the stored fp16
// coefficients; accumulation is fp32.
//
// Lane roles.  Lane (j, hf) = (lane % 32, lane / 32):
//   * as B operand it supplies atoms 8*hf .. 8*hf+7 of a 16-atom step for pixel
//     j, so lanes j and j+32 load different coefficient planes of the SAME
//     pixels: each lane loads PX consecutive pixels of a plane with one vector
//     load and re-packs (atom pair, pixel) with v_perm_b32;
//   * the MFMA result leaves pixel j's taps split over lanes j and j+32
//     (rows 8*(v/4) + 4*hf + v%4).  Dictionary rows are ordered so that half 0
//     owns filter rows 0 .. RH0-1 and half 1 owns rows RH0 .. (one dummy row
//     with zero weights): both halves then use the same LDS offsets, shifted by
//     RH0 tile rows.  Each half filters its taps against the LDS patch tile
//     and the two partial sums are exchanged across the halves.
//
// Software pipeline.  The atom steps are the outer loop and the PX pixel slots
// the inner one, so the registers of a step are free as soon as its MFMAs are
// issued: the same step of the NEXT tile is loaded into them right away.  The
// coefficient loads of tile t+1 are therefore in flight during stage 4 of tile
// t and during the up-sampling of tile t+1; the LR footprint is prefetched one
// tile ahead as well.
//
// The up-sampled tile is stored in LDS column-swizzled, (x % PX) major, so the
// 32 pixels of one MFMA (stride PX in x) read consecutive banks.
//
// Other coefficient types (template argument CT):
//   * CT_F32: 2-atom steps of v_mfma_f32_32x32x2_f32; lane half hf loads plane
//     2*step + hf and the loaded words are the B operand as they are; the
//     dictionary stays fp32, products and sums are true fp32;
//   * CT_F8 (8-bit E4M3 storage): 4 pixels per 4-byte load; the bytes of two planes
//     are paired per pixel with a byte permute and each pair is widened exactly to
//     the fp16 operand word, then the fp16 steps above;
//   * CT_BF16: the fp16 flow with the bfloat16 matrix instructions and the
//     dictionary as two bfloat16 operands;
//   * CT_LIST8 / CT_LIST16 (an extension beyond the paper): no planes, but per-pixel
//     lists of (atom, value) entries, scattered into the B operand through LDS
//     (see the constants below);
//   * CT_LOGIT / CT_LOGIT_BF16 (an extension beyond the paper): the planes hold logits and the
//     softmax over the atoms is part of the operand path (see the constants below).
// Other coefficient layouts (template argument PSM): the planes as the coefficient
// network holds them before its pixel-shuffle layer, pixel-major storage and the blocked
// order that needs no re-packing at all (see the kernel's own comment).
//
// Two forms of the walk over the image.  TILES (the original one, and the only one for the layouts before the pixel-shuffle and the
// blocked and pixel-major orders): a workgroup up-samples a tile and its halo into LDS in three barrier-separated steps, then its
// wavefronts fold and filter it.  STRIPS (template argument STRIP = the scale): a wavefront walks down its own segment of
// a strip of 32 PX columns; each row it up-samples one more row into a ring of K + 1 in its own LDS and folds, filters and stores one.  A row is
// up-sampled once per segment (not by every tile above and below it), neighbouring columns share their LR columns, the
// weights of the horizontal pass are compile-time constants, nothing waits at a barrier after the start, and the segments are cut to the
// number of wavefronts (a frame of 5.3 rounds of tiles takes six).  What bounded the light cases was exactly that: 4K with
// 8 of 72 atoms 79 -> 62 us (3.8 TB/s of a mix that is half writes), 4K lists of 8 141 -> 107, 4K fp8 154 -> 150, 720p fp8 33 -> 23, 4K fp16
// 248 -> 244, 4K logits 264 -> 253, four 7x7 video frames 409 -> 396; which form a call takes: strip_form().  Tried on top and not kept: two rows of
// coefficients in flight (registers spill, 62 -> 92 us), workgroups of 8 and 12 wavefronts that take half of each other's remaining
// rows (all wavefronts then end within 2 % instead of 15 %, and the call takes as long: the memory and the issue slots were busy before).
//
// L2 write-back pacing.  The output leaves the CUs as ordinary stores and sits in the XCDs' L2s as dirty lines that
// the L2 writes to memory when it sees fit, interleaved with the read stream; reads and writes that alternate at the
// memory cost more than their bytes (the stores of the 4K frame, 7.6 % of the bytes, cost 22 % of the time).  One
// wavefront per XCD (wavefront 0 of workgroups 0 .. 7, which the dispatcher deals to the eight XCDs) therefore asks
// its L2 every 16 us - by a constant-rate clock, checked once per unit - to write its dirty lines back NOW (an
// agent-scope release fence, which the compiler turns into the L2 write-back instruction and a wait): the writes
// reach memory in bursts and the reads in between run undisturbed.  Measured: 4K frame 254 -> 241 us, the blocked
// order 240 -> 231 us, 1080p 68 -> 65.5 us, sixteen video frames 1.80 -> 1.72 ms, 58 kept atoms 224 -> 215 us; neutral
// at 43 kept atoms and for 720p fp32, 1-2 % slower with fewer atoms and with 8-bit coefficients in tiles, which are not bound
// by the stream: those instantiations are launched without it.  The period was swept from 4 to 48 us (8 us and
// less cost time, beyond 32 us the gain fades; sixteen video frames of 7x7 atoms: 1.72 ms at 16 us, 1.69 at 24 to 32,
// hence 28 us there); results are bit-identical.  -DSR_NO_L2_WRITEBACK builds without it.
//
// Measurement builds (python -m paper_2303_08999_amd.build -o other.so -DSR_ABLATE_...): the
// same launch with a part switched off, to see what that part costs.  SR_ABLATE_STORES keeps
// every instruction but never executes the output stores; SR_ABLATE_STAGE1 skips the two
// up-sampling passes (barriers and LR rows stay); results are then wrong by construction.
// SR_STORES_WRITE_THROUGH writes the fp32 output of the four-pixel instantiations through the L2
// (agent scope) instead of leaving dirty lines in it; results are unchanged.
// The library built by default contains none of them.
#pragma once
#include <type_traits>

#include "sr_device.h"
#include "sr_launch.h"

namespace srd {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// how the coefficients are stored (template argument CT of the kernel)
constexpr int CT_F16 = 0, CT_F32 = 1, CT_F8 = 2, CT_BF16 = 3, CT_LIST8 = 4, CT_LIST16 = 5, CT_LOGIT = 6, CT_LOGIT_BF16 = 7;
// CT_LOGIT: the fp16 planes hold LOGITS (an extension beyond the paper, see sr_options.coeff_kind).  A unit's planes are
// loaded as in the fp16 form; once they are all there the lane takes the maximum of its pixels' logits (packed fp16
// maxima over its half of the planes, then one exchange with the other half), and where the fp16 form re-packs
// (atom pair, pixel) with a byte permute it forms exp2((z - max) log2 e) in fp32 - one mixed-precision
// multiply-add on the stored half and one exponential per value - and packs two of them, rounded to fp16, as the
// operand.  One padding row of the dictionary operand is all ones, so the matrix cores also return the sum of the
// exponentials of every pixel, in both lane halves; stage 4 multiplies its partial sums by the reciprocal.
// CT_LOGIT_BF16: bfloat16 logits.  The exponentials are fp16 operands all the same (11 significant bits, the range
// (0, 1]); a stored value is widened with a shift or a mask before the multiply-add.  The maxima are taken with the
// same packed fp16 instruction on the stored bits: sign, then magnitude bits, order bfloat16 values exactly as they
// order fp16 values, and the patterns that read as fp16 NaNs (bfloat16 magnitudes of 2^121 and up, the infinities
// among them) are passed over, which is what a logit of minus infinity, an atom switched off, asks for.
// CT_LIST8 / CT_LIST16: no dense planes; every pixel brings a list of up to 8 / 16 (atom index, fp16 value)
// entries (an extension beyond the paper, see sr_dict_assemble_list).  Each wavefront owns an LDS scratch
// [group of 8 atoms][32 pixels][8 atoms] fp16, all zero between uses.  Pixel slot by pixel slot it scatters
// the entries of 32 pixels into it (one 2-byte LDS write each; a lane writes only into its own pixel's 16-byte
// pieces, so few writes meet in a bank), reads its pieces back with 16-byte loads - the piece of group
// 2 c + hf is exactly the matrix cores' B operand of 16-atom step c in the dense form - and writes zeros where
// it wrote values.  The fold, the filtering and
// the store then run as for fp16 planes.
constexpr int LIST_MAX_ENTRIES = 16;

// SMIN: smallest scale the instantiation may be launched with.  The LR footprint
// of a tile shrinks with the scale, so an instantiation for scale 4 only needs half
// the LDS for the footprint and the vertical-pass buffer, and can afford a taller
// tile (fewer halo rows up-sampled per output row).
template <int K, int C, int NP8, int PX, int WR, int NW, int NU, int CT = CT_F16, int SMIN = 2, int NSUB = 1, int SWZ = 0, int STRIP = 0>
struct Cfg {
    static constexpr bool F32 = CT == CT_F32, F8 = CT == CT_F8, BF = CT == CT_BF16, LIST = CT == CT_LIST8 || CT == CT_LIST16;
    static constexpr bool LG = CT == CT_LOGIT || CT == CT_LOGIT_BF16, LGB = CT == CT_LOGIT_BF16;
    static constexpr int LH = CT == CT_LIST8 ? 4 : 8;  // list form: entries a lane half loads
    static constexpr int LSW = 4 * NP8 * 32;           // list form: scratch words per wavefront
    static constexpr int KK = K * K, R = (K - 1) / 2;
    static constexpr int RH0 = (K + 1) / 2;            // filter rows owned by lane half 0
    static constexpr int NSLOT = RH0 * K;              // accumulator rows used per half
    static constexpr int NMB = (NSLOT + 15) / 16;      // 32-row MFMA blocks
    static constexpr int WC = 32 / WR;                 // lane columns per wavefront
    static constexpr int TW = WC * PX * NSUB;          // tile of HR pixels per workgroup: NU units per wavefront, each
    static constexpr int TH = STRIP ? 1 : WR * NW * NU / NSUB;     // (strip form: a wavefront's own row) WR rows of WC * PX pixels; NSUB units share a row (see PSM = 4)
    static_assert(NU % NSUB == 0, "whole rows per wavefront");
    static constexpr int NT = 64 * NW;
    static constexpr int UW = TW + K - 1;
    static constexpr int UH = TH + K;                  // + one dummy row for half 1
    // The tile is stored column-swizzled: column x at (x % SW) * NG + x / SW, so that lanes whose columns are SW
    // apart read consecutive words.  SW = PX, except in the scale-4 pre-shuffle form (NSUB = 2), whose lane pairs
    // are 16 columns apart: with eight classes they step by two words, and the odd NG puts a pair's second lane on
    // the odd banks.
    // SWZ = 1 (pixel-major coefficients): no swizzle, lane j's slots are pixels j, 32 + j, ... of the row.
    static constexpr int SW = SWZ ? SWZ : (NSUB == 2 ? 8 : PX);
    static constexpr int NG = STRIP ? (UW + 3) / 4 * 4 / SW : ((UW + SW - 1) / SW) | (NSUB == 2 ? 1 : 0);   // stride between the classes
    static constexpr int P0 = SW * NG;
    // rows of one wavefront must land on disjoint banks: pitch == WC (mod 32)
    static constexpr int P = WR == 1 ? P0 : P0 + ((WC - P0 % 32) + 32) % 32;
    static constexpr int MAXLRY = (UH - 1) / SMIN + 5, MAXLRX = STRIP ? (UW + 1) / (STRIP ? STRIP : 1) + 6 : (UW - 1) / SMIN + 5;
    // Strip form: a wavefront's own LDS: a ring of SLOTS up-sampled rows, one row after the vertical pass, a ring of four LR rows
    static constexpr int SLOTS = 2 * RH0;
    static constexpr int LIT = (C * MAXLRX + 63) / 64, LROW = 64 * LIT;      // elements of an LR footprint row: per lane, and padded to whole wavefronts
    static constexpr int GPX = STRIP == 3 ? 3 : 4, GSTEP = STRIP == 2 ? 2 : 1;   // HR columns a lane up-samples at a time, their LR columns
    static constexpr int NGRP = STRIP == 3 ? (UW + 2 + 2) / 3 : (UW + 3) / 4, GIT = (C * NGRP + 63) / 64;
    static constexpr int WAVE_F = SLOTS * C * P + 5 * LROW;
    // fp16 coefficients: 16-atom MFMA steps and an optional 8-atom step;
    // fp32 coefficients: 2-atom steps of v_mfma_f32_32x32x2_f32, one load each
    static constexpr int N16 = F32 ? 0 : NP8 / 2, N8 = F32 ? 0 : NP8 % 2;
    static constexpr int N2 = F32 ? 4 * NP8 : 0;
    static constexpr int NLOAD = F32 ? N2 : (LIST ? 1 : 8 * N16 + 4 * N8);   // coefficient loads per lane and unit
    static constexpr int CB = F32 ? 4 : (F8 ? 1 : 2);  // bytes per stored coefficient
    static constexpr int NXC = (MAXLRX + 63) / 64;     // 64-column chunks of the LR footprint
    static constexpr int NLRP = (C * MAXLRY + NW - 1) / NW;   // (channel,row) pairs per wavefront
};

template <int BYTES> struct RawT;      // PX consecutive coefficients of one plane
template <> struct RawT<16> { typedef u32x4 type; };
template <> struct RawT<8> { typedef u32x2 type; };
template <> struct RawT<4> { typedef unsigned type; };

__device__ __forceinline__ unsigned raw_word(const u32x4& v, int m) { return v[m]; }
__device__ __forceinline__ unsigned raw_word(const u32x2& v, int m) { return v[m]; }
__device__ __forceinline__ unsigned raw_word(const unsigned& v, int) { return v; }

// Word m (fp16 pixels 2m, 2m+1) of one plane's raw load.  fp8 (e4m3) coefficients
// are widened here, two at a time; every e4m3 value is exact in fp16.
template <bool F8, int NWORD, typename RawV>
__device__ __forceinline__ void plane_words(const RawV& r, unsigned (&w)[NWORD]) {
    if constexpr (F8) {
        static_assert(NWORD == 2, "fp8 coefficients: four pixels per lane");
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        const unsigned bits = raw_word(r, 0);           // four fp8 pixels
        w[0] = __builtin_bit_cast(unsigned, (h2)__builtin_amdgcn_cvt_scalef32_pk_f16_fp8(bits, 1.0f, false));
        w[1] = __builtin_bit_cast(unsigned, (h2)__builtin_amdgcn_cvt_scalef32_pk_f16_fp8(bits, 1.0f, true));
    } else {
#pragma unroll
        for (int m = 0; m < NWORD; ++m) w[m] = raw_word(r, m);
    }
}

// 16- and 8-atom steps of the fold on packed 16-bit operands: fp16, or (BF) bfloat16
template <bool BF>
__device__ __forceinline__ f32x16 mfma_16(const u32x4& a, const u32x4& b, const f32x16& c) {
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <bool BF>
__device__ __forceinline__ f32x16 mfma_8(const u32x2& a, const u32x2& b, const f32x16& c) {
    if constexpr (BF)
        return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(f16x4, a), __builtin_bit_cast(f16x4, b), c, 0, 0, 0);
}
// Dictionary values as two 16-bit operands, d ~ hi + lo: 22 significant bits in fp16,
// 16 in bfloat16 (whose coefficients carry 8).
template <bool BF, int N, typename V>
__device__ __forceinline__ void split_hi_lo(const float (&d)[N], V& hi, V& lo) {
    unsigned short h[N], l[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        if constexpr (BF) {
            const __bf16 a = (__bf16)d[j];
            const __bf16 b = (__bf16)(d[j] - (float)a);
            h[j] = __builtin_bit_cast(unsigned short, a);
            l[j] = __builtin_bit_cast(unsigned short, b);
        } else {
            const _Float16 a = (_Float16)d[j];
            const _Float16 b = (_Float16)(d[j] - (float)a);
            h[j] = __builtin_bit_cast(unsigned short, a);
            l[j] = __builtin_bit_cast(unsigned short, b);
        }
    }
#pragma unroll
    for (int j = 0; j < N / 2; ++j) {
        hi[j] = (unsigned)h[2 * j] | ((unsigned)h[2 * j + 1] << 16);
        lo[j] = (unsigned)l[2 * j] | ((unsigned)l[2 * j + 1] << 16);
    }
}

// (atom pair, pixel q) from two planes' packed pixels
__device__ __forceinline__ unsigned pack_pair(unsigned plane_even, unsigned plane_odd, int q) {
    return __builtin_amdgcn_perm(plane_odd, plane_even, (q & 1) ? 0x07060302u : 0x05040100u);
}

// 8-bit coefficients: the four pixels of two planes as byte pairs (even plane, odd plane), pixels 0, 1 in w[0] and
// 2, 3 in w[1]; widen_pair then widens the pair of pixel q to the fp16 operand word (every E4M3 value is exact in fp16).
// Six instructions per plane pair where widening every plane first and pairing afterwards takes eight.
template <int NWORD>
__device__ __forceinline__ void pair_bytes(unsigned plane_even, unsigned plane_odd, unsigned (&w)[NWORD]) {
    static_assert(NWORD == 2, "8-bit coefficients: four pixels per lane");
    w[0] = __builtin_amdgcn_perm(plane_odd, plane_even, 0x05010400u);
    w[1] = __builtin_amdgcn_perm(plane_odd, plane_even, 0x07030602u);
}
__device__ __forceinline__ unsigned widen_pair(unsigned pairs, int q) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    return (q & 1) ? __builtin_bit_cast(unsigned, (h2)__builtin_amdgcn_cvt_scalef32_pk_f16_fp8(pairs, 1.0f, true))
                   : __builtin_bit_cast(unsigned, (h2)__builtin_amdgcn_cvt_scalef32_pk_f16_fp8(pairs, 1.0f, false));
}

// logits form: (atom pair, pixel q) as the exponentials exp2(z * log2(e) + nm) of the two planes' logits, rounded to fp16
// (BF16: the stored logits are bfloat16, the upper half of a binary32)
template <bool BF16>
__device__ __forceinline__ unsigned exp_pair(unsigned plane_even, unsigned plane_odd, int q, float nm) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    auto widen = [&](unsigned w) -> float {
        if constexpr (BF16) return __uint_as_float((q & 1) ? (w & 0xffff0000u) : (w << 16));
        else return (float)__builtin_bit_cast(h2, w)[q & 1];
    };
    const f2 e = {logit_exp(widen(plane_even), nm), logit_exp(widen(plane_odd), nm)};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(e, h2));      // round to nearest even
}
// ... of one word's two logits (blocked order: two atoms of one pixel side by side)
__device__ __forceinline__ unsigned exp_word(unsigned pair, float nm) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const h2 z = __builtin_bit_cast(h2, pair);
    const f2 e = {logit_exp((float)z[0], nm), logit_exp((float)z[1], nm)};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(e, h2));
}
// packed fp16 maximum of stored values (no canonicalising pass over the operands first)
__device__ __forceinline__ _Float16 __attribute__((ext_vector_type(2))) pk_max_f16(_Float16 __attribute__((ext_vector_type(2))) x,
                                                                                 _Float16 __attribute__((ext_vector_type(2))) y) {
    _Float16 __attribute__((ext_vector_type(2))) r;
    asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}

// Output stores through a raw buffer resource of the image (fourth word: 32-bit data format), whose bounds check drops a lane
// at the end of the image or beyond.  Such a lane stores up to eight bytes from the end on (or sixteen 64 bytes below 4 GB), and all of
// them have 32-bit offsets: every image below 4 GB, but fp32 ones of 2^30 - 1 pixels, whose pixel groups go in strips (see
// strip_form), where every lane is inside the image.
constexpr int RAW_BUFFER = 0x00020000;
__device__ __forceinline__ void store16(__amdgpu_buffer_rsrc_t r, unsigned at, float v) {
    __builtin_amdgcn_raw_buffer_store_b16(__half_as_ushort(narrow_f16(v)), r, at, 0, 0);
}
__device__ __forceinline__ void store32(__amdgpu_buffer_rsrc_t r, unsigned at, unsigned v) { __builtin_amdgcn_raw_buffer_store_b32(v, r, at, 0, 0); }
__device__ __forceinline__ void store64(__amdgpu_buffer_rsrc_t r, unsigned at, unsigned v0, unsigned v1) {
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{v0, v1}, r, at, 0, 0);
}
#ifdef SR_STORES_WRITE_THROUGH
constexpr int FP32_PAIR_POLICY = 16;                    // sc1: agent scope
#else
constexpr int FP32_PAIR_POLICY = 0;
#endif
__device__ __forceinline__ void store_fp32_pair(__amdgpu_buffer_rsrc_t r, unsigned at, float v0, float v1) {
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(v0), __float_as_uint(v1)}, r, at, 0, FP32_PAIR_POLICY);
}
__device__ __forceinline__ void store128(__amdgpu_buffer_rsrc_t r, unsigned at, const float (&v)[4]) {
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])}, r, at, 0, 0);
}
__device__ __forceinline__ unsigned pack_f16(float a, float b) {
    return (unsigned)__half_as_ushort(narrow_f16(a)) | ((unsigned)__half_as_ushort(narrow_f16(b)) << 16);
}

// filter tap served by MFMA row i of block mb, or -1 (padding / dummy row)
template <int K>
__device__ __forceinline__ int tap_of_row(int i, int mb) {
    constexpr int RH0 = (K + 1) / 2, NSLOT = RH0 * K;
    const int half = (i >> 2) & 1;
    const int vv = 16 * mb + (((i >> 3) << 2) | (i & 3));
    if (vv >= NSLOT) return -1;
    const int dy = half * RH0 + vv / K, dx = vv % K;
    return dy < K ? dy * K + dx : -1;
}

// logits form: the MFMA row (one per lane half) that is all ones: the first padding row of the block that holds it
template <int K>
__device__ __forceinline__ bool sum_row(int i, int mb) {
    constexpr int NSLOT = ((K + 1) / 2) * K;
    return 16 * mb + (((i >> 3) << 2) | (i & 3)) == NSLOT;
}

struct TilePos { int n, ty, tx; };

// v = q * s + r, 0 <= r < s, for the scales the library takes (wave-uniform branch on s)
__device__ __forceinline__ void divmod_scale(int v, int s, int& q, int& r) {
    if (s == 4) { q = v >> 2; r = v & 3; }
    else if (s == 2) { q = v >> 1; r = v & 1; }
    else { q = v / 3; r = v - 3 * q; }
}

// PSM != 0: the coefficients are read in the layout the coefficient network holds before its
// pixel-shuffle layer, [L*s*s][h][w]: the s*s sub-pixels of an LR pixel lie in s*s LR planes.
//   PSM = 4 (scale 4) and PSM = 2 (scale 2): the fast forms.  Which HR pixel an MFMA column and
//     pixel slot stand for is free, as long as stage 4 and the store know it.  A lane still loads
//     8 bytes per plane, but from ONE sub-pixel plane: four consecutive LR pixels, i.e. four HR
//     pixels s apart, which become its four slots.  With n = lane % 32, j = n % 2, m = n / 2:
//       scale 2: the lane reads sub-pixel column j;  slot q is HR pixel X0 + 8 m + 2 q + j.
//         A unit is one row of 128 HR pixels = 64 LR pixels = one 128-byte line of each plane.
//       scale 4: 128 HR pixels of a row would be half a line of each plane, and a half-line
//         request occupies the L1 like a whole one (measured: the same bytes in 64-byte pieces
//         take 2.2 x the time unless the same wavefront asks for the other half right away).  So the
//         tile is 256 pixels wide and a row is TWO units, J = 0, 1: the lane reads sub-pixel column
//         2 J + j;  slot q is HR pixel X0 + 16 m + 4 q + 2 J + j.  Every load instruction still
//         covers whole lines (16 lanes x 8 bytes per plane).
//       scale 3: the tile is 384 pixels wide and a row is THREE units, J = 0, 1, 2: every lane reads
//         sub-pixel column J, lane n the LR columns 4 n .. 4 n + 3;  slot q is HR pixel X0 + 12 n + 3 q + J
//         (two whole lines of a plane per lane half).  No exchange before the store: after the third
//         unit a lane holds six adjacent pixels.
//     Loads are as many and as wide as in the HR-planar form.  Stage 4 reads the tile at those
//     pixels (per-lane LDS bases), and before the store lanes j = 0, 1 exchange results so that
//     each holds adjacent pixels again (scale 4: the results of unit J = 0 wait in registers for
//     J = 1, then a lane stores four adjacent pixels and a wavefront 1 KB per channel).
//   PSM = 1 (any scale): the PX consecutive HR pixels of a lane come from up to PX planes, one
//     16-bit load each, placed in the halves of the registers an HR-planar load would have
//     filled; everything after the loads is unchanged.  Four times the load instructions and a
//     register per element in flight: 2.6 x the time of the planar form at 4K.
// The result is the planar form's, bit for bit, in every case.
//
// PSM = 8: the coefficients are stored pixel-major, [H][W][L] (the L = 72 coefficients of a pixel side by
// side, 144 bytes; what a producer that keeps its tensors channels-last writes).  A unit's 128 pixels are
// then 18 432 CONTIGUOUS bytes: 18 loads of 16 bytes per lane, lane after lane (the friendliest request
// stream there is: the same bytes take 231 us where the planes take 249).  Sixteen bytes of a pixel are the
// eight atoms of half a 16-atom step, i.e. a B operand as it stands: pixel slot by pixel slot (slot q =
// pixels 32 q .. 32 q + 31 of the unit, 4 608 contiguous bytes) the loaded registers are copied to an LDS
// scratch as they are and lane (j, hf) reads its operand pieces back at pixel j, piece 2 c + hf.  No
// re-packing.  Lane j's slots are the pixels j, 32 + j, 64 + j, 96 + j: the tile is stored without a
// swizzle (consecutive lanes read consecutive words) and a lane stores single pixels (a wavefront half
// still writes 128 contiguous bytes).  The fold, stage 4 and the result are the planar form's, bit for bit.
//
// PSM = 9: the coefficients are stored BLOCKED (SR_COEFF_BLOCKED; a storage order beyond the paper, for a producer that
// is willing to write it): a unit's 128 x 72 coefficients are 18 432 contiguous bytes laid out as this kernel consumes
// them - slot q (pixel 4 j + q of the unit), then pieces of 16 atoms [lane half][column j][8 atoms] and a last piece
// [lane half][column j][4 atoms].  Lane (j, hf) = lane j + 32 hf loads 16 bytes at 16 * lane of a piece (a wavefront: 1 KB
// of contiguous memory per load) and holds the B operand of that 16-atom step and slot as it stands: no re-packing, no
// staging, and the slots are the planar form's four adjacent pixels, so stage 4 and the store are the planar form's too.
// (8-bit coefficients in the same order: 8 bytes per lane and piece, widened to the operand with four conversions.)
// KEEP: coefficient loads leave their lines in the caches (see keep_lines).
template <int K, int C, int NP8, int PX, int WR, int NW, int NU, int WPE, int CT, int SMIN, bool BIG, int PSM = 0, int STRIP = 0, bool KEEP = false>
__global__ __launch_bounds__(64 * NW, WPE)
void k_assemble_mfma(const AssembleArgs a) {
    constexpr int NSUB = PSM == 4 ? 2 : (PSM == 3 ? 3 : 1);   // units per tile row
    constexpr bool PMAJ = PSM == 8;                // coefficients stored pixel-major, [H][W][L]
    constexpr bool BLK = PSM == 9;                 // coefficients stored blocked: the loaded registers are the operands
    using F = Cfg<K, C, NP8, PX, WR, NW, NU, CT, SMIN, NSUB, (PMAJ ? 1 : 0), STRIP>;
    static_assert(!STRIP || (WR == 1 && NU == 1 && PSM == 0 && !BIG), "strip form: one row of a wavefront's strip at a time");
    constexpr bool F32 = F::F32, F8 = F::F8, BF = F::BF, LIST = F::LIST, LG = F::LG;
    static_assert(!LG || (PX == 4 && (PSM == 0 || PSM == 2 || PSM == 3 || PSM == 4 || PSM == 9) && !BIG && F::NSLOT < 16 * F::NMB),
                  "logits form: fp16 planes (or the permuted-slot forms of the layout before the pixel-shuffle), four pixels per lane, a free MFMA row");
    constexpr int LH = F::LH;                      // list entries a lane half loads
    static_assert(!LIST || (PX == 4 && WR == 1 && !BIG && PSM == 0 && (STRIP != 0 || NU % 2 == 0)), "list form: four pixels per lane, one row per unit");
    constexpr bool PS = PSM == 1;                  // one 16-bit load per pixel
    constexpr bool PERM = PSM == 2 || PSM == 3 || PSM == 4;    // permuted pixel slots
    static_assert(PSM == 0 || ((CT == CT_F16 || (CT == CT_F8 && PSM == 9) ||
                                ((CT == CT_BF16 || CT == CT_LOGIT || CT == CT_LOGIT_BF16) && PSM != 1 && PSM != 8 &&
                                 (PSM != 9 || CT == CT_LOGIT || CT == CT_BF16))) && !BIG && PX == 4),
                  "pre-shuffle layout: 16-bit coefficients, four pixels per lane");
    static_assert(!PMAJ || (CT == CT_F16 && WR == 1 && NP8 == 9), "pixel-major coefficients: 72 fp16 atoms, one row per unit");
    static_assert(!BLK || ((CT == CT_F16 || CT == CT_BF16 || CT == CT_F8 || CT == CT_LOGIT) && WR == 1 && PX == 4),
                  "blocked coefficients: fp16 (values or logits), bfloat16 or 8-bit, one row of 128 pixels per unit");
    static_assert(!PERM || (WR == 1 && SMIN >= PSM), "permuted slots: one row per wavefront and unit");
    // row of the wavefront's unit within the tile, and which of the row's NSUB units it is
    auto unit_row = [](int unit, int wave_) { return STRIP ? 0 : (unit / NSUB) * NW + wave_; };
    constexpr int NPIX = PS ? PX : 1;              // pixel offsets a lane keeps per unit
    using Raw = typename RawT<PX * F::CB>::type;
    constexpr int NT = F::NT, P = F::P, NG = F::NG, UH = F::UH, UW = F::UW;
    constexpr int N16 = F::N16, N8 = F::N8, NMB = F::NMB;
    constexpr int MAXLRY = F::MAXLRY, MAXLRX = F::MAXLRX;

    __shared__ float U[STRIP ? NW * F::WAVE_F : C * UH * P];   // up-sampled tile, column-swizzled (strip form: all of a wavefront's buffers)
    __shared__ float V[STRIP ? 1 : C * UH * MAXLRX];           // after the vertical pass
    __shared__ float lrT[STRIP ? 1 : C * MAXLRY * MAXLRX];     // LR footprint (clamped reads)
    __shared__ float4 xw[STRIP ? 1 : UW], yw[STRIP ? 1 : UH];  // per-column / per-row tap weights
    __shared__ int xb[STRIP ? 1 : UW], yb[STRIP ? 1 : UH];     // ... and first source index
    __shared__ float4 wk[8];                        // Keys weights by phase numerator m
    __shared__ u32x4 A16[(N16 ? N16 : 1) * NMB * 2 * 64];
    __shared__ u32x2 A8[(F32 ? 1 : NMB * 2) * 64];
    __shared__ float A32[(F32 ? F::N2 * NMB : 1) * 64];   // fp32 path: D[2*step + hf][tap of row]
    __shared__ unsigned ptab[2 * F::NLOAD];         // byte offset of the plane each lane half loads
    __shared__ u32x4 pmscr[PMAJ ? NW * 288 : 1];    // pixel-major: per wavefront, one slot's 32 pixels x 144 bytes
    __shared__ unsigned ltab[LIST ? 2 * LH : 1];    // list form: element offset of the entry plane each lane half loads
    __shared__ u32x4 lscr[LIST ? NW * F::LSW / 4 : 1];   // list form: per wavefront, [NP8 groups of 8 atoms][32 pixels][8 atoms] fp16

    const int tid0 = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);     // scalar, loop-invariant
    const int tiles_x = a.tiles_x, tiles_y = a.tiles_y, G = a.stride;
    const int grp = (int)blockIdx.x & ((1 << a.group_shift) - 1);
    const int t_end = min(a.ntiles, (grp + 1) * a.share);
    const int t_block = grp * a.share + ((int)blockIdx.x >> a.group_shift) * (STRIP ? NW : 1);
    if (t_block >= t_end) return;                                  // whole workgroup: no tile
    // (strip form: a "tile" is a segment of a strip and belongs to one wavefront; one past the end loads what the last one
    //  loads and does nothing with it)
    const int t_first = STRIP ? t_block + wave : t_block;
    // First column of a tile.  When the image width is not a whole number of pixel
    // groups the last tile column is moved left to end at the image edge (a.xlast =
    // W - TW): it recomputes some pixels of its neighbour (same values, written twice)
    // and no lane ever holds a group that sticks out of its row.
    auto tile_x0 = [&](int tx) { return tx == tiles_x - 1 ? a.xlast : tx * F::TW; };

    // ---- once per workgroup: weight, plane-offset and dictionary operand tables ---
    // Where a coefficient lies within its image is a 32-bit offset: in bytes, or (BIG) in
    // elements, which reaches images of up to 2^32 coefficients (an 8K frame with 72 fp16
    // planes is 4.8 GB) at the price of a 64-bit address per load instead of a scalar base
    // plus a 32-bit offset.
    constexpr unsigned OU = BIG ? 1u : (unsigned)F::CB;                          // offset units per element
    const unsigned plane_b = (unsigned)a.H * (unsigned)a.W * OU;                 // offset units per coefficient plane
    auto caddr = [&](const char* img, unsigned off) -> const char* {
        if constexpr (BIG) return img + (size_t)off * (size_t)F::CB;
        else return img + off;
    };
    if constexpr (LIST) {
        for (int e = tid0; e < NW * F::LSW / 4; e += NT) lscr[e] = u32x4{0u, 0u, 0u, 0u};
        // half h takes entries h * ceil(T / 2) ...; a slot past the list repeats an entry the pixel has (the
        // half's first one, or entry 0): written twice to the same place with the same value
        const int per_half = (a.T + 1) / 2;
        for (int e = tid0; e < 2 * LH; e += NT) {
            const int h = e / LH, i = e - h * LH;
            int t = h * per_half + i;
            if (i >= per_half || t >= a.T) t = h * per_half < a.T ? h * per_half : 0;
            ltab[e] = (unsigned)t * ((unsigned)a.H * (unsigned)a.W);               // in elements
        }
    }
    // Folded atom that load i of lane half h serves; the table of plane offsets (padding atoms re-read the last plane)
    auto load_atom = [&](int i, int h) -> int {
        return F32 ? 2 * i + h : (i < 8 * N16 ? 16 * (i >> 3) + 8 * h + (i & 7) : 16 * N16 + 4 * h + (i - 8 * N16));
    };
    // What bounds the start of a launch is latency: each step that waits for memory, and each scalar load of another line
    // of the kernel arguments, costs up to 1 us, and a launch used to spend 3.4 to 5.7 us before its first coefficient was
    // requested (list and scales, then the dictionary entry by entry behind a branch, six divisions).  Now the dictionary's
    // entries are requested first, all of them, unconditionally (clamped addresses; what is padding becomes zero at
    // its use), then the LR footprint and the first unit's coefficients, and only then is anything waited for.  The whole
    // dictionary in its own order (a.identity) needs no look at the list; a kept list goes through LDS once.
    __shared__ int ktab[LIST ? 1 : 8 * NP8];        // first dictionary element of a folded atom
    __shared__ float gtab[LIST ? 1 : 8 * NP8];      // its scale
    if (!LIST && !a.identity) {
        for (int e = tid0; e < 8 * NP8; e += NT) {
            const int i = e < a.n_fold ? e : a.n_fold - 1;
            const int k = a.kept[i];
            const float g = a.gamma[i];
            ktab[e] = k * F::KK;
            gtab[e] = g;
        }
        __syncthreads();
    }
    for (int e = tid0; e < (LIST ? 0 : 2 * F::NLOAD); e += NT) {
        const int h = e / F::NLOAD, at = load_atom(e - h * F::NLOAD, h);
        ptab[e] = (unsigned)(a.identity ? (at < a.n_fold ? at : a.n_fold - 1) : ktab[at] / F::KK) * plane_b;
    }
    // A wavefront makes whole blocks of 64 lanes of the dictionary operands: block b of a kind is that of wavefront b % NW.
    const int lane0 = tid0 & 63, half0 = lane0 >> 5;
    const bool whole = LIST || a.identity;
    auto dict_entry = [&](int at, int tap) -> float {
        const int row = whole ? (at < a.n_fold ? at : a.n_fold - 1) * F::KK : ktab[at];
        return a.dict[(unsigned)(row + (tap < 0 ? 0 : tap))];
    };
    auto dict_value = [&](int at, int tap, float d) -> float {              // gamma * D[kept], zero for padding
        const float g = whole ? 1.0f : gtab[at];
        return tap < 0 || at >= a.n_fold ? 0.0f : g * d;
    };
    constexpr int NB32 = F32 ? F::N2 * NMB : 0, NB16 = N16 * NMB, NB8 = N8 ? NMB : 0;     // blocks of each kind
    constexpr int M32 = (NB32 + NW - 1) / NW, M16 = (NB16 + NW - 1) / NW, M8 = (NB8 + NW - 1) / NW;   // ... of a wavefront
    float dv32[M32 ? M32 : 1];
    float dv16[M16 ? M16 : 1][8], dv8[M8 ? M8 : 1][4];
#pragma unroll
    for (int m = 0; m < M32; ++m) {
        const int blk = wave + NW * m < NB32 ? wave + NW * m : NB32 - 1, mb = blk % NMB, st = blk / NMB;
        dv32[m] = dict_entry(2 * st + half0, tap_of_row<K>(lane0 & 31, mb));
    }
#pragma unroll
    for (int m = 0; m < M16; ++m) {
        const int blk = wave + NW * m < NB16 ? wave + NW * m : NB16 - 1, mb = blk % NMB, c16 = blk / NMB;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj)
            dv16[m][jj] = dict_entry(16 * c16 + 8 * half0 + jj, tap_of_row<K>(lane0 & 31, mb));
    }
#pragma unroll
    for (int m = 0; m < M8; ++m) {
        const int mb = wave + NW * m < NB8 ? wave + NW * m : NB8 - 1;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
            dv8[m][jj] = dict_entry(16 * N16 + 4 * half0 + jj, tap_of_row<K>(lane0 & 31, mb));
    }
    __builtin_amdgcn_sched_barrier(0);
    // ... and into LDS once they are there (with the up-sampling weights, by phase)
    auto store_operands = [&]() {
        if (tid0 < 2 * a.s) {
            float wt[4];
            keys_weights(tid0, a.s, wt);
            wk[tid0] = make_float4(wt[0], wt[1], wt[2], wt[3]);
        }
#pragma unroll
        for (int m = 0; m < M32; ++m) {
            const int blk = wave + NW * m, mb = blk % NMB, st = blk / NMB;
            if (blk < NB32) A32[blk * 64 + lane0] = dict_value(2 * st + half0, tap_of_row<K>(lane0 & 31, mb), dv32[m]);
        }
#pragma unroll
        for (int m = 0; m < M16; ++m) {
            const int blk = wave + NW * m, mb = blk % NMB, c16 = blk / NMB;
            if (blk < NB16) {
                const int tap = tap_of_row<K>(lane0 & 31, mb);
                const bool ones = LG && sum_row<K>(lane0 & 31, mb);   // logits form: this row sums the exponentials
                float dv[8];
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) {
                    const int at = 16 * c16 + 8 * half0 + jj;
                    dv[jj] = ones ? (at < a.n_fold ? 1.0f : 0.0f) : dict_value(at, tap, dv16[m][jj]);
                }
                u32x4 hi, lo;
                split_hi_lo<BF, 8>(dv, hi, lo);
                A16[(blk * 2 + 0) * 64 + lane0] = hi;
                A16[(blk * 2 + 1) * 64 + lane0] = lo;
            }
        }
#pragma unroll
        for (int m = 0; m < M8; ++m) {
            const int mb = wave + NW * m;
            if (mb < NB8) {
                const int tap = tap_of_row<K>(lane0 & 31, mb);
                const bool ones = LG && sum_row<K>(lane0 & 31, mb);
                float dv[4];
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int at = 16 * N16 + 4 * half0 + jj;
                    dv[jj] = ones ? (at < a.n_fold ? 1.0f : 0.0f) : dict_value(at, tap, dv8[m][jj]);
                }
                u32x2 hi, lo;
                split_hi_lo<BF, 4>(dv, hi, lo);
                A8[(mb * 2 + 0) * 64 + lane0] = hi;
                A8[(mb * 2 + 1) * 64 + lane0] = lo;
            }
        }
    };

    // ---- tile walk.  Workgroups are dealt to the 8 XCDs round-robin by index, and
    //      each XCD has its own L2.  When the grid is a multiple of 8, XCD x (the
    //      workgroups with blockIdx.x % 8 == x) walks its own contiguous share of the
    //      tiles in raster order, so that tiles above one another, whose LR
    //      footprints overlap, meet in the same L2 at about the same time.  The
    //      step is pre-split into (image, tile row, tile column) so that no
    //      division is left in the loop.  All of it is scalar.
    const int step_n = a.step_n, step_y = a.step_y, step_x = a.step_x;
    auto advance = [&](TilePos p) -> TilePos {
        p.tx += step_x;
        if (p.tx >= tiles_x) { p.tx -= tiles_x; p.ty += 1; }
        p.ty += step_y;
        if (p.ty >= tiles_y) { p.ty -= tiles_y; p.n += 1; }
        p.n += step_n;
        return p;
    };
    // quotients by the rounded-down reciprocals are at most one too small (0 <= t < 2^31)
    auto tile_of = [&](int t) -> TilePos {
        TilePos p;
        p.n = (int)(((unsigned long long)(unsigned)t * a.inv_img) >> 32);
        int r = t - p.n * a.per_img;
        if (r >= a.per_img) { r -= a.per_img; p.n += 1; }
        p.ty = (int)(((unsigned long long)(unsigned)r * a.inv_tx) >> 32);
        p.tx = r - p.ty * tiles_x;
        if (p.tx >= tiles_x) { p.tx -= tiles_x; p.ty += 1; }
        return p;
    };
    TilePos cur = tile_of(STRIP ? min(t_first, t_end - 1) : t_first);

    const char* lr_base = (const char*)a.lr;
    const unsigned lr_esz = a.io_f16 ? 2u : 4u;

    // LR footprint of a tile -> registers, as raw bits (fp16 is widened when it is
    // written to LDS).  Wavefront w takes (channel,row) pairs w, w+NW, ...; the lane
    // is the column.  Row addressing is scalar; one add per load on the vector side.
    //
    // Two forms.  LRBF (used where the coefficient stream is light enough for the
    // issue time of these loads to show, measured 4 % on the 8-bit 4K frame): every
    // slot is loaded unconditionally, as the aligned 32-bit word holding the
    // element (an fp16 image keeps which half in `par`, one bit per slot); slots
    // the tile does not need repeat the wavefront's first row / chunk, a line that
    // is already on its way.  No branch and one load type leave the compiler
    // nothing to merge at a join, so the loads go out back to back.  Otherwise:
    // only the needed slots are loaded (fewer requests, which is what counts when
    // the stream is the bound or the tile is small).
    constexpr bool LRBF = F8 && NP8 > 2;
    static_assert(!LRBF || F::NLRP * F::NXC <= 32, "one parity bit per footprint slot");
    const unsigned lr_sh = a.io_f16 ? 1u : 2u;          // log2 of the element size
    auto load_lr = [&](const TilePos tp, int lane, unsigned (&lrv)[F::NLRP][F::NXC], unsigned& par) {
        const TileOrigin o = tile_origin(tp.ty * F::TH, tile_x0(tp.tx), F::R, UH, UW, a.H, a.W, a.s);
        // the image's base is a 64-bit scalar; offsets within an image fit 32 bits
        const char* lr_img = lr_base + (size_t)tp.n * C * ((size_t)a.h * a.w * lr_esz);
        if constexpr (LRBF) {
            // aligned words: the image may start in the middle of one
            const unsigned mis = (unsigned)((uintptr_t)lr_img & 3u);
            const char* lr_al = lr_img - mis;
            unsigned xcol[F::NXC];
#pragma unroll
            for (int xc = 0; xc < F::NXC; ++xc) {
                xcol[xc] = (unsigned)clampi(o.lx0 + lane + 64 * xc, 0, a.w - 1);
                if (xc > 0 && 64 * xc >= o.nlx) xcol[xc] = xcol[0];
            }
            par = 0u;
            unsigned row0 = 0u;
#pragma unroll
            for (int u = 0; u < F::NLRP; ++u) {
                const int p = wave + NW * u, c = p / MAXLRY, ry = p - c * MAXLRY;
                const bool need = p < C * MAXLRY && ry < o.nly;
                unsigned row = ((unsigned)(need ? c : 0) * (unsigned)a.h +
                                (unsigned)clampi(o.ly0 + (need ? ry : 0), 0, a.h - 1)) * (unsigned)a.w;   // in elements
                if (u == 0) row0 = row;
                if (!need) row = row0;
#pragma unroll
                for (int xc = 0; xc < F::NXC; ++xc) {
                    const unsigned byte = ((row + xcol[xc]) << lr_sh) + mis;
                    par |= ((byte >> 1) & 1u) << (u * F::NXC + xc);
                    lrv[u][xc] = *(const unsigned*)(lr_al + (size_t)(byte & ~3u));
                }
            }
        } else {
            unsigned xo[F::NXC];
#pragma unroll
            for (int xc = 0; xc < F::NXC; ++xc) xo[xc] = (unsigned)clampi(o.lx0 + lane + 64 * xc, 0, a.w - 1) * lr_esz;
            auto rows = [&](auto f16) {
#pragma unroll
                for (int u = 0; u < F::NLRP; ++u) {
                    const int p = wave + NW * u, c = p / MAXLRY, ry = p - c * MAXLRY;
                    if (p < C * MAXLRY && ry < o.nly) {
                        const unsigned row = ((unsigned)c * (unsigned)a.h +
                                              (unsigned)clampi(o.ly0 + ry, 0, a.h - 1)) * (unsigned)a.w * lr_esz;
#pragma unroll
                        for (int xc = 0; xc < F::NXC; ++xc)
                            if (xc == 0 || 64 * xc < o.nlx) {     // whole 64-column chunks the tile never reads
                                const char* q = lr_img + (size_t)(row + xo[xc]);
                                lrv[u][xc] = decltype(f16)::value ? (unsigned)*(const unsigned short*)q : *(const unsigned*)q;
                            }
                    }
                }
            };
            if (a.io_f16) rows(std::true_type{});
            else rows(std::false_type{});
        }
    };

    // coefficient base of a tile for this lane: image base (scalar) + pixel offset
    auto phi_base = [&](const TilePos tp, int unit, int jr, int jc, unsigned (&pix_off)[NPIX]) -> const char* {
        const int y = tp.ty * F::TH + unit_row(unit, wave) * WR + jr, x = tile_x0(tp.tx) + PX * jc;
        const int yc = y < a.H ? y : a.H - 1, xc = x < a.W ? x : a.W - PX;   // out-of-image lanes re-read
        if constexpr (PERM) {
            // jc is the lane's column n: sub-pixel column (unit % NSUB) * 2 + n % 2, LR columns 4 m .. 4 m + 3, m = n / 2
            // (scale 3: every lane reads sub-pixel column unit % 3, lane n the LR columns 4 n .. 4 n + 3)
            const int jx = PSM == 3 ? unit % NSUB : (unit % NSUB) * 2 + jc % 2, m = PSM == 3 ? jc : jc / 2;
            const int ly = yc / PSM, iy = yc % PSM;
            int lx = tile_x0(tp.tx) / PSM + 4 * m;
            lx = lx + 4 <= a.w ? lx : a.w - 4;                                     // lanes past the image re-read
            pix_off[0] = ((unsigned)(iy * PSM + jx) * ((unsigned)a.h * (unsigned)a.w) +
                          (unsigned)ly * (unsigned)a.w + (unsigned)lx) * OU;
        } else if constexpr (PS) {
            int ly, iy;
            divmod_scale(yc, a.s, ly, iy);
            const unsigned hw = (unsigned)a.h * (unsigned)a.w;
#pragma unroll
            for (int q = 0; q < PX; ++q) {
                int lx, jx;
                divmod_scale(xc + q, a.s, lx, jx);
                pix_off[q] = ((unsigned)(iy * a.s + jx) * hw + (unsigned)ly * (unsigned)a.w + (unsigned)lx) * OU;
            }
        } else {
            pix_off[0] = ((unsigned)yc * (unsigned)a.W + (unsigned)xc) * OU;         // a valid address; never stored
        }
        return (const char*)a.coeff + (size_t)tp.n * a.L * ((size_t)a.H * a.W * F::CB);
    };
    // the PX coefficients of one plane (or plane group) that a lane owns
    auto load_raw = [&](const char* cimg, const unsigned (&pix_off)[NPIX], unsigned plane_off) -> Raw {
        if constexpr (PS) {
            typedef _Float16 h2 __attribute__((ext_vector_type(2)));
            Raw r;
#pragma unroll
            for (int m = 0; m < PX / 2; ++m) {
                h2 v;
                v[0] = __builtin_nontemporal_load((const _Float16*)(cimg + (pix_off[2 * m] + plane_off)));
                v[1] = __builtin_nontemporal_load((const _Float16*)(cimg + (pix_off[2 * m + 1] + plane_off)));
                r[m] = __builtin_bit_cast(unsigned, v);
            }
            return r;
        } else {
            const Raw* const at = (const Raw*)caddr(cimg, pix_off[0] + plane_off);
            if constexpr (KEEP) return *at;
            else return __builtin_nontemporal_load(at);
        }
    };

    // list form: the entries of a unit, two register sets (the next unit's are loaded while this one is folded)
    u32x2 lval[2][LIST ? LH : 1];                   // four fp16 values (the lane's four pixels) per entry
    unsigned lidx[2][LIST ? LH : 1];                // their four atom numbers, one byte each
    // (img: elements before the image's first; pix: the lane's pixels within a plane)
    auto load_list_at = [&](size_t img, unsigned pix, int hf, u32x2 (&val)[LIST ? LH : 1], unsigned (&idx)[LIST ? LH : 1]) {
        const unsigned char* ibase = a.index + img;
        const char* vbase = (const char*)a.coeff + img * 2;
        const unsigned* lt = ltab + hf * LH;
#pragma unroll
        for (int e = 0; e < LH; ++e) {
            const unsigned at = lt[e] + pix;
            idx[e] = __builtin_nontemporal_load((const unsigned*)(ibase + at));
            val[e] = __builtin_nontemporal_load((const u32x2*)(vbase + (size_t)at * 2));
        }
    };
    auto load_list = [&](const TilePos tp, int unit, int jc, int hf, u32x2 (&val)[LIST ? LH : 1], unsigned (&idx)[LIST ? LH : 1]) {
        const int y = tp.ty * F::TH + unit_row(unit, wave), x = tile_x0(tp.tx) + PX * jc;
        const int yc = y < a.H ? y : a.H - 1, xc = x < a.W ? x : a.W - PX;
        load_list_at((size_t)tp.n * a.T * ((size_t)a.H * a.W), (unsigned)yc * (unsigned)a.W + (unsigned)xc, hf, val, idx);
    };
    // pixel-major: the unit's 18 432 bytes, 16 per lane and load; byte offset of the lane's first piece within the image
    constexpr int NPM = 18;
    u32x4 pm[PMAJ ? NPM : 1];
    auto pm_offset = [&](const TilePos tp, int unit, int lane_) -> unsigned {
        const int y = tp.ty * F::TH + unit * NW + wave;
        const unsigned yc = (unsigned)(y < a.H ? y : a.H - 1);                 // rows past the image re-read its last row
        return (yc * (unsigned)a.W + (unsigned)tile_x0(tp.tx)) * (unsigned)(16 * NP8) + 16u * (unsigned)lane_;
    };
    auto pm_image = [&](const TilePos tp) -> const char* {
        return (const char*)a.coeff + (size_t)tp.n * a.L * ((size_t)a.H * a.W * F::CB);
    };
    // blocked: byte offset of a unit within its image (a unit: 128 pixels x 8 NP8 atoms, contiguous), and its loads
    // (8-bit coefficients: the same order of elements, half the bytes: 8 bytes per lane and 16-atom piece, widened to the
    //  operand at its use)
    using B16 = typename std::conditional<F8, u32x2, u32x4>::type;
    using B8 = typename std::conditional<F8, unsigned, u32x2>::type;
    constexpr unsigned CBB = (unsigned)F::CB;
    B16 b16[BLK ? PX : 1][BLK && N16 ? N16 : 1];
    B8 b8[BLK ? PX : 1];
    constexpr unsigned SLOT_B = 32u * 8u * NP8 * CBB;   // bytes of a slot: 32 pixels x 8 NP8 atoms
    auto blk_offset = [&](const TilePos tp, int unit) -> unsigned {
        const int y = tp.ty * F::TH + unit * NW + wave;
        const unsigned yc = (unsigned)(y < a.H ? y : a.H - 1);                 // rows past the image re-read its last row
        return (yc * (unsigned)(a.W / 128) + (unsigned)tp.tx) * (4u * SLOT_B);
    };
    auto blk_load16 = [&](const char* img, unsigned unit_off, int lane_, int q, int c16) -> B16 {
        return __builtin_nontemporal_load((const B16*)(img + (unit_off + (unsigned)q * SLOT_B + 512u * CBB * c16 + 8u * CBB * lane_)));
    };
    auto blk_load8 = [&](const char* img, unsigned unit_off, int lane_, int q) -> B8 {
        return __builtin_nontemporal_load((const B8*)(img + (unit_off + (unsigned)q * SLOT_B + 512u * CBB * N16 + 4u * CBB * lane_)));
    };
    // an 8-atom run of 8-bit coefficients widened to the fp16 operand (exact), two values per conversion
    auto widen16 = [&](const u32x2& v) -> u32x4 {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        u32x4 r;
#pragma unroll
        for (int m = 0; m < 4; ++m)
            r[m] = (m & 1) ? __builtin_bit_cast(unsigned, (h2)__builtin_amdgcn_cvt_scalef32_pk_f16_fp8(v[m >> 1], 1.0f, true))
                           : __builtin_bit_cast(unsigned, (h2)__builtin_amdgcn_cvt_scalef32_pk_f16_fp8(v[m >> 1], 1.0f, false));
        return r;
    };
    auto widen8 = [&](unsigned v) -> u32x2 {
        typedef _Float16 h2 __attribute__((ext_vector_type(2)));
        u32x2 r;
        r[0] = __builtin_bit_cast(unsigned, (h2)__builtin_amdgcn_cvt_scalef32_pk_f16_fp8(v, 1.0f, false));
        r[1] = __builtin_bit_cast(unsigned, (h2)__builtin_amdgcn_cvt_scalef32_pk_f16_fp8(v, 1.0f, true));
        return r;
    };
    // ---- strip form (STRIP = the scale): a wavefront walks down a segment of a strip of TW columns, row by row.  Its
    //      up-sampled rows live in an LDS ring of its own (K rows, and the one that the second lane half reads against zero
    //      weights): every row is up-sampled once per segment instead of once per tile that touches it, there is no barrier after
    //      the start, and a lane's four (scale 3: three) neighbouring columns share their LR columns and have compile-time weights.
    constexpr int S_ = STRIP ? STRIP : 4;
    if constexpr (STRIP != 0) cur.ty *= a.seg_rows;     // `cur`: image, image row, strip
    constexpr int LIT = STRIP ? F::LIT : 1, LROW = F::LROW;
    float* const ring = U + (STRIP ? wave * F::WAVE_F : 0);
    float* const vrow = ring + F::SLOTS * C * P;        // a row after the vertical pass: [channel][LR column]
    float* const lring = vrow + LROW;                   // four LR rows
    unsigned soff[LIT], sinit[4][LIT], spre[LIT];       // byte offset of the lane's elements in an LR row; raw LR rows on their way
    int sfloor = 0, sshift = 0;                         // LR row sfloor + 2 is the last in the ring, sfloor + 3 is in spre
    unsigned sread[STRIP ? F::GIT : 1], swrite[STRIP ? F::GIT : 1];   // a lane's groups of columns: first LR column in vrow, place in a ring row
    const char* simg = lr_base;
    auto strip_fence = []() {                           // other lanes' LDS writes: ordered by the hardware, and here for the compiler
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto strip_load = [&](int ly, unsigned (&v)[LIT], const auto io_f16) {
        const char* row = simg + (size_t)clampi(ly, 0, a.h - 1) * ((size_t)a.w * lr_esz);
        if (io_f16) {
#pragma unroll
            for (int i = 0; i < LIT; ++i) v[i] = (unsigned)*(const unsigned short*)(row + soff[i]);
        } else {
#pragma unroll
            for (int i = 0; i < LIT; ++i) v[i] = *(const unsigned*)(row + soff[i]);
        }
    };
    auto strip_store = [&](int ly, const unsigned (&v)[LIT], int lane, const auto io_f16) {
#pragma unroll
        for (int i = 0; i < LIT; ++i)
            lring[(ly & 3) * LROW + lane + 64 * i] = io_f16 ? __half2float(__ushort_as_half((unsigned short)v[i])) : __uint_as_float(v[i]);
    };
    // a segment's first five LR rows are requested ... (sg.ty: its first row)
    auto strip_begin = [&](const TilePos sg, int lane, const auto io_f16) {
        const int X0 = tile_x0(sg.tx), xr = X0 - F::R;
        sshift = STRIP == 3 ? (xr + 3) % 3 : 0;         // scale 3: groups start at a column that is a multiple of 3
        const int f0 = (2 * (xr - sshift) + 1 - S_ + 4 * S_) / (2 * S_) - 2;
        simg = lr_base + (size_t)sg.n * C * ((size_t)a.h * a.w * lr_esz);
#pragma unroll
        for (int i = 0; i < LIT; ++i) {
            const int e = lane + 64 * i < C * MAXLRX ? lane + 64 * i : C * MAXLRX - 1, c = e / MAXLRX, rx = e - c * MAXLRX;
            soff[i] = ((unsigned)c * (unsigned)a.h * (unsigned)a.w + (unsigned)clampi(f0 - 1 + rx, 0, a.w - 1)) * lr_esz;
        }
#pragma unroll
        for (int i = 0; i < F::GIT; ++i) {
            const int e = lane + 64 * i < C * F::NGRP ? lane + 64 * i : C * F::NGRP - 1, c = e / F::NGRP, g = e - c * F::NGRP;
            sread[i] = c * MAXLRX + g * F::GSTEP;
            swrite[i] = c * P + (STRIP == 3 ? 0 : g * (4 / F::SW));
        }
        int m;
        sfloor = src_floor_s<S_>(clampi(sg.ty - F::R, 0, a.H - 1), m);
#pragma unroll
        for (int i = 0; i < 4; ++i) strip_load(sfloor - 1 + i, sinit[i], io_f16);
        strip_load(sfloor + 3, spre, io_f16);
    };
    // Row Y + 1 of the up-sampled image is begun and row Y finished (rows outside the image: its first and last).  Both
    // passes' LDS reads go out together: the horizontal pass of Y, from what the vertical one left in vrow, into ring slot
    // `slot` (not if that is negative), and the vertical pass of Y + 1.
    auto strip_rows = [&](int Y, int slot, const TilePos sg, int lane, const auto io_f16) {
        int m;
        const int f = src_floor_s<S_>(clampi(Y + 1, 0, a.H - 1), m);
        strip_fence();
        if (f != sfloor) {                              // by one: the next LR row
            strip_store(sfloor + 3, spre, lane, io_f16);
            sfloor = f;
            strip_load(f + 3, spre, io_f16);
            strip_fence();
        }
#ifdef SR_ABLATE_STAGE1
        if (a.N >= 0) return;
#endif
        constexpr int PH = STRIP == 3 ? 0 : (F::R / S_ + 1) * S_ - F::R;     // a column with the phase of a group's first
        constexpr int NV = 4 + (F::GPX - 1 + S_ - 1) / S_;                   // (at most that many LR columns)
        float v[F::GIT][NV], r[LIT][4];
#pragma unroll
        for (int i = 0; i < F::GIT; ++i)
#pragma unroll
            for (int j = 0; j < NV; ++j) v[i][j] = vrow[sread[i] + j];
        const float4 w4 = wk[m];
#pragma unroll
        for (int i = 0; i < LIT; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) r[i][j] = lring[((f - 1 + j) & 3) * LROW + lane + 64 * i];
        strip_fence();
        if (slot >= 0) {
            float* const dst = ring + slot * (C * P);
            int mp;
            const int fp = src_floor_s<S_>(PH, mp);
#pragma unroll
            for (int i = 0; i < F::GIT; ++i)
#pragma unroll
                for (int q = 0; q < F::GPX; ++q) {
                    int mq;
                    const int d = src_floor_s<S_>(PH + q, mq) - fp;
                    float wq[4];
                    keys_weights(mq, S_, wq);
                    const float u = dot4(wq, v[i][d], v[i][d + 1], v[i][d + 2], v[i][d + 3]);
                    if constexpr (STRIP == 3) {
                        const int e = lane + 64 * i < C * F::NGRP ? lane + 64 * i : C * F::NGRP - 1;
                        const int xx = 3 * (e % F::NGRP) + q - sshift;
                        if (xx >= 0 && xx < UW) dst[swrite[i] + (xx % F::SW) * NG + xx / F::SW] = u;
                    } else {
                        dst[swrite[i] + (q % F::SW) * NG + q / F::SW] = u;
                    }
                }
            // columns outside the image are copies of its first and last column (a strip that starts at a column from 1 to R - 1 would
            // need them on the left too: not launched, see strip_form)
            const int X0 = tile_x0(sg.tx);
            if (X0 == 0 || X0 + F::TW + F::R > a.W) {
                strip_fence();
                int le = lane;                          // (these few addresses are not worth registers held over the rows)
                asm volatile("" : "+v"(le));
                const int side = le / (C * F::R), c = le / F::R % C, i = le % F::R;
                const int from = side == 0 ? F::R : a.W - 1 - X0 + F::R, to = side == 0 ? i : a.W - X0 + F::R + i;
                if (side == 0 ? X0 == 0 : side == 1 && to < UW)
                    dst[c * P + (to % F::SW) * NG + to / F::SW] = dst[c * P + (from % F::SW) * NG + from / F::SW];
            }
        }
        const float wv[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
        for (int i = 0; i < LIT; ++i) vrow[lane + 64 * i] = dot4(wv, r[i][0], r[i][1], r[i][2], r[i][3]);
    };
    // the next row's coefficients (image, the lane's offset in it) and this row's output, from row to row
    const char* snext = nullptr;
    char* sout = nullptr;
    unsigned spix = 0u, so0 = 0u;
    size_t slist = 0;
    // this form's loads of few planes take their offsets from registers
    constexpr bool PTREG = STRIP != 0 && !LIST && F::NLOAD <= 4;
    unsigned preg[PTREG ? F::NLOAD : 1];
    Raw raw[F::NLOAD];
    unsigned lrv[F::NLRP][F::NXC], lrpar = 0u;
#pragma unroll
    for (int u = 0; u < F::NLRP; ++u)
#pragma unroll
        for (int xc = 0; xc < F::NXC; ++xc) lrv[u][xc] = 0u;
    {
        const int lane = tid0 & 63, hf = lane >> 5, j = lane & 31;
        if constexpr (STRIP != 0) strip_begin(cur, lane, a.io_f16);
        else load_lr(cur, lane, lrv, lrpar);
        if constexpr (LIST) {
            __syncthreads();                            // ltab is written
            load_list(cur, 0, j, hf, lval[0], lidx[0]);
        } else if constexpr (PMAJ) {
            const char* img = pm_image(cur);
            const unsigned off = pm_offset(cur, 0, lane);
#pragma unroll
            for (int i = 0; i < NPM; ++i) pm[i] = __builtin_nontemporal_load((const u32x4*)(img + (off + 1024u * i)));
        } else if constexpr (BLK) {
            const char* img = pm_image(cur);
            const unsigned off = blk_offset(cur, 0);
#pragma unroll
            for (int q = 0; q < PX; ++q) {
#pragma unroll
                for (int c16 = 0; c16 < N16; ++c16) b16[q][c16] = blk_load16(img, off, lane, q, c16);
                if constexpr (N8 != 0) b8[q] = blk_load8(img, off, lane, q);
            }
        } else {
            unsigned pix_off[NPIX];
            const char* cimg = phi_base(cur, 0, j / F::WC, j % F::WC, pix_off);
            if (a.identity && a.n_fold == 8 * NP8) {
                // load i's planes are the half's first plane plus a whole number of planes: the scalar base walks
                const char* pl = cimg;
                const unsigned half_b = hf ? plane_b : 0u;
#pragma unroll
                for (int i = 0; i < F::NLOAD; ++i) {
                    const unsigned first = F32 ? half_b : (i < 8 * N16 ? 8u * half_b : 4u * half_b);
                    raw[i] = load_raw(pl, pix_off, first);
                    if (i + 1 < F::NLOAD) pl = caddr(pl, plane_b) + (size_t)(load_atom(i + 1, 0) - load_atom(i, 0) - 1) * plane_b * (BIG ? F::CB : 1);
                }
            } else {
                __syncthreads();                        // the table of plane offsets is written
                const unsigned* pt = ptab + hf * F::NLOAD;
#pragma unroll
                for (int i = 0; i < F::NLOAD; ++i) raw[i] = load_raw(cimg, pix_off, pt[i]);
            }
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    store_operands();
    __syncthreads();

    // list form with up to 72 atoms, and pixel-major coefficients: the dictionary operands stay in registers (the
    // fold reads them once per pixel slot, four times as often as the dense form does)
    constexpr bool AREG = (LIST && NP8 <= 9) || PSM == 8;
    u32x4 areg[AREG ? 2 * N16 : 1];
    u32x2 areg8[AREG && N8 ? 2 : 1];
    if constexpr (AREG) {
#pragma unroll
        for (int i = 0; i < 2 * N16; ++i) {
            areg[i] = A16[i * 64 + (tid0 & 63)];
            asm volatile("" : "+v"(areg[i]));           // opaque: or the compiler reloads it from LDS at every use
        }
        if constexpr (N8 != 0) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                areg8[i] = A8[i * 64 + (tid0 & 63)];
                asm volatile("" : "+v"(areg8[i]));
            }
        }
    }


    // ---- stage 1 in three steps; a workgroup barrier separates each from the next.
    // (a) tap tables of a tile and its LR footprint, registers -> LDS
    // the first UW threads fill the column tables, UH of the last 64 the row tables
    static_assert(UH <= 64, "tile too tall for the table set-up");
    auto stage1_setup = [&](const TilePos tp, int tid) {
        const int lane = tid & 63;
        const int Y0 = tp.ty * F::TH, X0 = tile_x0(tp.tx);
        const TileOrigin o = tile_origin(Y0, X0, F::R, UH, UW, a.H, a.W, a.s);
        for (int xx = tid; xx < UW; xx += NT) {       // one pass unless the tile is wider than the workgroup
            int m;
            const int f = src_floor(clampi(X0 - F::R + xx, 0, a.W - 1), a.s, m);
            xw[xx] = wk[m];
            xb[xx] = clampi(f - 1 - o.lx0, 0, MAXLRX - 4);
        }
        if (tid >= NT - 64 && tid - (NT - 64) < UH) {
            const int i = tid - (NT - 64);
            int m;
            const int f = src_floor(clampi(Y0 - F::R + i, 0, a.H - 1), a.s, m);
            yw[i] = wk[m];
            yb[i] = clampi(f - 1 - o.ly0, 0, MAXLRY - 4);
        }
#pragma unroll
        for (int u = 0; u < F::NLRP; ++u) {
            const int p = wave + NW * u;
            if (p < C * MAXLRY) {
#pragma unroll
                for (int xc = 0; xc < F::NXC; ++xc)
                    if (lane + 64 * xc < MAXLRX) {
                        unsigned bits = lrv[u][xc];
                        if (LRBF && a.io_f16) bits = ((lrpar >> (u * F::NXC + xc)) & 1u) ? bits >> 16 : bits & 0xffffu;
                        lrT[p * MAXLRX + lane + 64 * xc] =
                            a.io_f16 ? __half2float(__ushort_as_half((unsigned short)bits)) : __uint_as_float(bits);
                    }
            }
        }
    };
    // (b) vertical pass on the narrow LR footprint: V[c][yy][rx].  Four elements per
    //     thread at a time, their table reads and then their 16 footprint reads
    //     issued together, so that LDS latency is paid once per batch and not twice
    //     per element.  Loads are clamped into range; only the store is guarded.
    auto stage1_vertical = [&](const TilePos tp, int tid) {
        const TileOrigin o = tile_origin(tp.ty * F::TH, tile_x0(tp.tx), F::R, UH, UW, a.H, a.W, a.s);
        // Items (row pr, footprint column rx), nlx columns to a row, dealt to the threads with
        // no idle lanes (rows padded to 32, 64 or 128 columns left 38 % of them idle at x4:
        // 8 atoms at 4K 90 -> 85 us, the E4M3 frame 160 -> 154 us).  idx / nlx by a multiply,
        // exact for idx < 2^22 / nlx and free of overflow for idx < 1024 nlx.
        static_assert(C * UH * MAXLRX * MAXLRX <= (1 << 22) && C * UH <= 1024, "item index beyond the exact range of the division");
        const int nlx = o.nlx < 4 ? 4 : o.nlx;
        const unsigned inv = ((1u << 22) + nlx - 1) / nlx;
        const int total = C * UH * nlx;
        for (int base = tid; base < total; base += 4 * NT) {
            float4 w4[4];
            int src[4], dst[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int idx = base + k * NT;
                const int idc = idx < total ? idx : total - 1;
                const int pr = (int)(((unsigned)idc * inv) >> 22), rx = idc - pr * nlx;
                const int c = pr / UH, yy = pr - c * UH;
                w4[k] = yw[yy];
                src[k] = (c * MAXLRY + yb[yy]) * MAXLRX + rx;
                dst[k] = idx < total ? pr * MAXLRX + rx : -1;
            }
            __builtin_amdgcn_sched_barrier(0);
            float v[4][4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[k][i] = lrT[src[k] + i * MAXLRX];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float wt[4] = {w4[k].x, w4[k].y, w4[k].z, w4[k].w};
                if (dst[k] >= 0) V[dst[k]] = dot4(wt, v[k][0], v[k][1], v[k][2], v[k][3]);
            }
        }
    };
    // (c) horizontal pass into the swizzled tile: a thread owns one (channel,
    //     column), its weights stay in registers, rows are independent (no tables,
    //     immediate offsets).  Rows go in batches: all reads of a batch are issued
    //     before its arithmetic.
    auto stage1_horizontal = [&](int tid) {
        for (int col = tid; col < C * UW; col += NT) {
            const int c = col / UW, xx = col - c * UW;
            const float4 w4 = xw[xx];
            const float wt[4] = {w4.x, w4.y, w4.z, w4.w};
            const float* src = V + c * UH * MAXLRX + xb[xx];
            float* dst = U + c * UH * P + (xx % F::SW) * NG + xx / F::SW;
            constexpr int RB = 7;
#pragma unroll
            for (int y0 = 0; y0 < UH; y0 += RB) {
                float v[RB][4];
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    if (y0 + r < UH) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[r][i] = src[(y0 + r) * MAXLRX + i];
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    if (y0 + r < UH) dst[(y0 + r) * P] = dot4(wt, v[r][0], v[r][1], v[r][2], v[r][3]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    float park[C][NSUB > 1 ? NSUB - 1 : 1][2];         // permuted slots, scales 3 and 4: the results of a row's earlier units wait for the last
    unsigned long long wb_last = a.wb_ticks > 0 ? __builtin_amdgcn_s_memrealtime() : 0ull;
    // A unit: stage 3, stage 4 and the store of WR rows of WC * PX pixels; `more_tiles`: the unit after the tile's last is unit 0 of `nxt`.
    // (slot0: strip form, ring slot of the first filter row; more_tiles and io_f16: booleans, or the types of known ones)
    auto do_unit = [&](const int unit, const TilePos here, const TilePos nxt, const auto more_tiles, const int tid, const int slot0,
                       const auto io_f16) __attribute__((always_inline)) {
        const int lane = tid & 63;
        const int hf = lane >> 5, j = lane & 31, jr = j / F::WC, jc = j % F::WC;
        const int Y0 = here.ty * F::TH, X0 = tile_x0(here.tx);
        const unsigned* pt = ptab + hf * F::NLOAD;
        const bool last_unit = STRIP || unit == NU - 1;
        const bool more = last_unit ? (bool)more_tiles : true;
        unsigned pix_next[NPIX];
        const char* cnext = nullptr;
        if constexpr (STRIP != 0 && !BLK) {
            pix_next[0] = spix;
            cnext = snext;
        } else if constexpr (!LIST && !PMAJ && !BLK) cnext = last_unit ? phi_base(nxt, 0, jr, jc, pix_next) : phi_base(here, unit + 1, jr, jc, pix_next);
        const char* bimg = nullptr;                    // blocked: the next unit's image and offset
        unsigned boff = 0u;
        if constexpr (BLK) {
            bimg = last_unit ? pm_image(nxt) : pm_image(here);
            boff = last_unit ? blk_offset(nxt, 0) : blk_offset(here, unit + 1);
        }

        // (3) stage 3 on the matrix cores: atom steps outer, pixel slots inner
        f32x16 acc[PX][NMB];
#pragma unroll
        for (int q = 0; q < PX; ++q)
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[q][mb][v] = 0.0f;
        if constexpr (LIST) {
            // the next unit's entries go into the other register set while this one is folded
            if (more) {
                if constexpr (STRIP != 0) load_list_at(slist, spix, hf, lval[(unit + 1) & 1], lidx[(unit + 1) & 1]);
                else if (last_unit) load_list(nxt, 0, jc, hf, lval[(unit + 1) & 1], lidx[(unit + 1) & 1]);
                else load_list(here, unit + 1, jc, hf, lval[(unit + 1) & 1], lidx[(unit + 1) & 1]);
            }
            const u32x2 (&val)[LH] = lval[unit & 1];
            const unsigned (&idx)[LH] = lidx[unit & 1];
            static_assert(NMB == 1, "list form: one block of MFMA rows");
            // (16-bit writes and vector reads of the same words: the write goes through a type that may alias
            //  anything, or the compiler is free to move a read above the write it depends on)
            typedef unsigned short __attribute__((may_alias)) u16a;
            u32x4* const scrw = lscr + wave * (F::LSW / 4);
            char* const col = (char*)(scrw + jc);              // atom a of the lane's pixel: col + (a / 8) * 512 + (a % 8) * 2
            // Per pixel slot: scatter, read the operand pieces, write the zeros back - all three go out at once
            // (LDS serves a wavefront's requests in order) - and only the fold waits for the pieces.  The next
            // slot's requests are issued before this slot's fold, so that they travel while the matrix cores work.
            u32x4 bw16[2][N16 ? N16 : 1];
            u32x2 bw8[2];
            auto issue = [&](int q, int b) {
                // lanes j and j + 32 hold different entries of the same pixels.  An atom number the dictionary
                // does not have (a caller's error) is kept inside the pixel's own pieces.
                unsigned where[LH];
#pragma unroll
                for (int e = 0; e < LH; ++e) {
                    unsigned atom = (idx[e] >> (8 * q)) & 0xffu;
                    atom = atom < 8u * NP8 ? atom : 8u * NP8 - 1u;
                    where[e] = (atom >> 3) * 512u + (atom & 7u) * 2u;
                    *(u16a*)(col + where[e]) = (unsigned short)(val[e][q >> 1] >> (16 * (q & 1)));
                }
#pragma unroll
                for (int c16 = 0; c16 < N16; ++c16) bw16[b][c16] = scrw[(2 * c16 + hf) * 32 + jc];
                if constexpr (N8 != 0) bw8[b] = *(const u32x2*)(col + (2 * N16) * 512 + 8 * hf);
#pragma unroll
                for (int e = 0; e < LH; ++e) *(u16a*)(col + where[e]) = (unsigned short)0;
            };
            issue(0, 0);
#pragma unroll
            for (int q = 0; q < PX; ++q) {
                __builtin_amdgcn_sched_barrier(0);
                if (q + 1 < PX) issue(q + 1, (q + 1) & 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c16 = 0; c16 < N16; ++c16)
#pragma unroll
                    for (int hl = 0; hl < 2; ++hl)
                        acc[q][0] = mfma_16<false>(AREG ? areg[c16 * 2 + hl] : A16[(c16 * 2 + hl) * 64 + lane], bw16[q & 1][c16], acc[q][0]);
                if constexpr (N8 != 0) {
#pragma unroll
                    for (int hl = 0; hl < 2; ++hl)
                        acc[q][0] = mfma_8<false>(AREG ? areg8[hl] : A8[hl * 64 + lane], bw8[q & 1], acc[q][0]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (PMAJ) {
            static_assert(NMB == 1 || !PMAJ, "pixel-major: one block of MFMA rows");
            const char* nimg = last_unit ? pm_image(nxt) : pm_image(here);
            const unsigned noff = last_unit ? pm_offset(nxt, 0, lane) : pm_offset(here, unit + 1, lane);
            char* const scr = (char*)(pmscr + wave * 288);
            const char* const mine = scr + jc * (16 * NP8);            // the lane's pixel of the slot
            auto reload = [&](int i) {
                if (more) pm[i] = __builtin_nontemporal_load((const u32x4*)(nimg + (noff + 1024u * i)));
            };
            // Slot q = stream bytes 4608 q .. 4608 q + 4607: four whole loads and half of the load that two slots
            // share.  stage(q): registers -> scratch (and the freed registers are re-loaded for the next unit), then
            // the lane's operand pieces back: sixteen bytes of a pixel are atoms 8 g .. 8 g + 7, piece 2 c + hf is
            // the operand of step c.  LDS serves a wavefront's requests in order, so the next slot is staged
            // before this slot's matrix instructions are issued and its pieces travel while they run.
            u32x4 bw16[2][N16 ? N16 : 1];
            u32x2 bw8[2];
            auto stage = [&](int q, int b) {
                const int first = (9 * q) / 2;                         // 0, 4, 9, 13
                if (q % 2 == 0) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) *(u32x4*)(scr + 1024 * i + 16 * lane) = pm[first + i];
                    if (lane < 32) *(u32x4*)(scr + 4096 + 16 * lane) = pm[first + 4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) reload(first + i);
                } else {
                    if (lane >= 32) *(u32x4*)(scr + 16 * (lane - 32)) = pm[first];
#pragma unroll
                    for (int i = 0; i < 4; ++i) *(u32x4*)(scr + 512 + 1024 * i + 16 * lane) = pm[first + 1 + i];
#pragma unroll
                    for (int i = 0; i < 5; ++i) reload(first + i);
                }
#pragma unroll
                for (int c16 = 0; c16 < N16; ++c16) bw16[b][c16] = *(const u32x4*)(mine + 32 * c16 + 16 * hf);
                if constexpr (N8 != 0) bw8[b] = *(const u32x2*)(mine + 32 * N16 + 8 * hf);
            };
            stage(0, 0);
#pragma unroll
            for (int q = 0; q < PX; ++q) {
                __builtin_amdgcn_sched_barrier(0);
                if (q + 1 < PX) stage(q + 1, (q + 1) & 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c16 = 0; c16 < N16; ++c16)
#pragma unroll
                    for (int hl = 0; hl < 2; ++hl)
                        acc[q][0] = mfma_16<false>(AREG ? areg[c16 * 2 + hl] : A16[(c16 * 2 + hl) * 64 + lane], bw16[q & 1][c16], acc[q][0]);
                if constexpr (N8 != 0) {
#pragma unroll
                    for (int hl = 0; hl < 2; ++hl)
                        acc[q][0] = mfma_8<false>(AREG ? areg8[hl] : A8[hl * 64 + lane], bw8[q & 1], acc[q][0]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (F32) {
            // fp32 coefficients: the loaded words ARE the B operand (lane half hf holds
            // atom 2*step + hf of its pixels), no re-packing, exact fp32 products
#pragma unroll
            for (int st = 0; st < F::N2; ++st) {
                float av[NMB];
#pragma unroll
                for (int mb = 0; mb < NMB; ++mb) av[mb] = A32[(st * NMB + mb) * 64 + lane];
#pragma unroll
                for (int q = 0; q < PX; ++q)
#pragma unroll
                    for (int mb = 0; mb < NMB; ++mb)
                        acc[q][mb] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                            av[mb], __uint_as_float(raw_word(raw[st], q)), acc[q][mb], 0, 0, 0);
                if ((st & 3) == 3) __builtin_amdgcn_sched_barrier(0);
                if (more)
                    raw[st] = load_raw(cnext, pix_next, PTREG ? preg[PTREG ? st : 0] : pt[st]);
                if ((st & 3) == 3) __builtin_amdgcn_sched_barrier(0);
            }
        }
        // logits form: -max * log2(e) of the lane's four pixels, over all planes (both lane halves)
        float nm[PX];
        if constexpr (LG && BLK) {
            // blocked order: a word holds two atoms of ONE pixel (slot q); per slot the packed maximum over the lane's
            // words, the larger of its two halves, then the other lane half's
            typedef _Float16 h2 __attribute__((ext_vector_type(2)));
#pragma unroll
            for (int q = 0; q < PX; ++q) {
                const unsigned first = N16 ? b16[q][0][0] : b8[q][0];
                h2 mq = __builtin_bit_cast(h2, first);
#pragma unroll
                for (int c16 = 0; c16 < N16; ++c16)
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const unsigned word = b16[q][c16][m];       // (by value: a bit cast straight from the vector element read element 0)
                        mq = pk_max_f16(mq, __builtin_bit_cast(h2, word));
                    }
                if constexpr (N8 != 0) {
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        const unsigned word = b8[q][m];
                        mq = pk_max_f16(mq, __builtin_bit_cast(h2, word));
                    }
                }
                const unsigned bits = __builtin_bit_cast(unsigned, mq);
                mq = pk_max_f16(mq, __builtin_bit_cast(h2, (bits >> 16) | (bits << 16)));       // both halves: the larger one
                const unsigned one = __builtin_bit_cast(unsigned, mq);
                const auto sw = __builtin_amdgcn_permlane32_swap(one, one, false, false);
                mq = pk_max_f16(__builtin_bit_cast(h2, (unsigned)sw[0]), __builtin_bit_cast(h2, (unsigned)sw[1]));
                nm[q] = logit_shift((float)mq[0]);
            }
        } else if constexpr (LG) {
            typedef _Float16 h2 __attribute__((ext_vector_type(2)));
            h2 mx[PX / 2];
#pragma unroll
            for (int m = 0; m < PX / 2; ++m) mx[m] = __builtin_bit_cast(h2, raw_word(raw[0], m));
#pragma unroll
            for (int i = 1; i < F::NLOAD; ++i)
#pragma unroll
                for (int m = 0; m < PX / 2; ++m) mx[m] = pk_max_f16(mx[m], __builtin_bit_cast(h2, raw_word(raw[i], m)));
#pragma unroll
            for (int m = 0; m < PX / 2; ++m) {
                const unsigned bits = __builtin_bit_cast(unsigned, mx[m]);
                const auto sw = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);   // one of the two is the other half's
                mx[m] = pk_max_f16(__builtin_bit_cast(h2, (unsigned)sw[0]), __builtin_bit_cast(h2, (unsigned)sw[1]));
            }
#pragma unroll
            for (int q = 0; q < PX; ++q) {
                if constexpr (F::LGB) nm[q] = logit_shift(__uint_as_float((__builtin_bit_cast(unsigned, mx[q >> 1]) >> (16 * (q & 1))) << 16));
                else nm[q] = logit_shift((float)mx[q >> 1][q & 1]);
            }
        }
#pragma unroll
        for (int c16 = 0; c16 < (LIST || PMAJ ? 0 : N16); ++c16) {   // (the list and pixel-major forms have folded above)
            u32x4 av[NMB][2];
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                for (int hl = 0; hl < 2; ++hl) av[mb][hl] = A16[((c16 * NMB + mb) * 2 + hl) * 64 + lane];
            constexpr int NWORD = PX / 2 > 0 ? PX / 2 : 1;
            unsigned cw[8][NWORD];                  // the step's 8 planes as fp16 pixel pairs
            if constexpr (BLK) {
                // (blocked: the loaded registers are the operands)
            } else if constexpr (F8) {
                // 8-bit coefficients: pair the planes' BYTES first (two permutes per plane pair), widen afterwards
#pragma unroll
                for (int m = 0; m < 4; ++m) pair_bytes(raw_word(raw[8 * c16 + 2 * m], 0), raw_word(raw[8 * c16 + 2 * m + 1], 0), cw[2 * m]);
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) plane_words<F8>(raw[8 * c16 + i], cw[i]);
            }
#pragma unroll
            for (int q = 0; q < PX; ++q) {
                u32x4 bw;
                if constexpr (BLK) {
                    if constexpr (F8) bw = widen16(b16[q][c16]);
                    else if constexpr (LG) {
#pragma unroll
                        for (int m = 0; m < 4; ++m) bw[m] = exp_word(b16[q][c16][m], nm[q]);
                    } else bw = b16[q][c16];
                }
#pragma unroll
                for (int m = 0; m < (BLK ? 0 : 4); ++m)
                    bw[m] = F8 ? widen_pair(cw[2 * m][q >> 1], q)
                          : LG ? exp_pair<F::LGB>(cw[2 * m][q >> 1], cw[2 * m + 1][q >> 1], q, nm[q])
                               : pack_pair(cw[2 * m][q >> 1], cw[2 * m + 1][q >> 1], q);
#pragma unroll
                for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                    for (int hl = 0; hl < 2; ++hl) acc[q][mb] = mfma_16<BF>(av[mb][hl], bw, acc[q][mb]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (more) {
                if constexpr (BLK) {
#pragma unroll
                    for (int q = 0; q < PX; ++q) b16[q][c16] = blk_load16(bimg, boff, lane, q, c16);
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        raw[8 * c16 + i] = load_raw(cnext, pix_next, PTREG ? preg[PTREG ? 8 * c16 + i : 0] : pt[8 * c16 + i]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (N8 != 0 && !LIST && !PMAJ) {
            u32x2 av[NMB][2];
#pragma unroll
            for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                for (int hl = 0; hl < 2; ++hl) av[mb][hl] = A8[(mb * 2 + hl) * 64 + lane];
            constexpr int NWORD = PX / 2 > 0 ? PX / 2 : 1;
            unsigned cw[4][NWORD];
            if constexpr (BLK) {
            } else if constexpr (F8) {
#pragma unroll
                for (int m = 0; m < 2; ++m) pair_bytes(raw_word(raw[8 * N16 + 2 * m], 0), raw_word(raw[8 * N16 + 2 * m + 1], 0), cw[2 * m]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) plane_words<F8>(raw[8 * N16 + i], cw[i]);
            }
#pragma unroll
            for (int q = 0; q < PX; ++q) {
                u32x2 bw;
                if constexpr (BLK) {
                    if constexpr (F8) bw = widen8(b8[q]);
                    else if constexpr (LG) {
#pragma unroll
                        for (int m = 0; m < 2; ++m) bw[m] = exp_word(b8[q][m], nm[q]);
                    } else bw = b8[q];
                }
#pragma unroll
                for (int m = 0; m < (BLK ? 0 : 2); ++m)
                    bw[m] = F8 ? widen_pair(cw[2 * m][q >> 1], q)
                          : LG ? exp_pair<F::LGB>(cw[2 * m][q >> 1], cw[2 * m + 1][q >> 1], q, nm[q])
                               : pack_pair(cw[2 * m][q >> 1], cw[2 * m + 1][q >> 1], q);
#pragma unroll
                for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                    for (int hl = 0; hl < 2; ++hl) acc[q][mb] = mfma_8<BF>(av[mb][hl], bw, acc[q][mb]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (more) {
                if constexpr (BLK) {
#pragma unroll
                    for (int q = 0; q < PX; ++q) b8[q] = blk_load8(bimg, boff, lane, q);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        raw[8 * N16 + i] = load_raw(cnext, pix_next, PTREG ? preg[PTREG ? 8 * N16 + i : 0] : pt[8 * N16 + i]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }

        // (4) stage 4: each half filters its taps against the LDS tile, channel by
        //     channel (a lane's PX slots share most of their patch values)
        const float* ub = U + (unit_row(unit, wave) * WR + jr + hf * F::RH0) * P + (PERM ? 0 : jc);
        // Permuted slots: slot q, tap dx reads tile column G m + e0 + j, with G = 8 or 16 (two groups of SW = 4 or 8
        // columns) and the compile-time e0 = 2 q + dx (scale 2) or 4 q + 2 J + dx (scale 4).  The swizzled index
        // of a column x is (x % SW) NG + x / SW.  The lane's j enters through two per-lane bases, so that every
        // read is base + immediate offset: e0 % SW < SW - 1: class e0 % SW + j of the same group; otherwise the
        // last class, or (j = 1) class 0 of the next group.
        unsigned ubo[2] = {0u, 0u};                    // as element offsets into U
        if constexpr (PMAJ) {
            // column 32 q + j + dx of an unswizzled tile: the lane enters as j
            ubo[0] = ubo[1] = (unsigned)((unit_row(unit, wave) * WR + jr + hf * F::RH0) * P + jc);
        }
        if constexpr (PERM) {
            const int jx = jc % 2, m = jc / 2;
            const int row0 = (unit_row(unit, wave) * WR + jr + hf * F::RH0) * P;
            if constexpr (PSM == 3) {
                // column 12 n + 3 q + J + dx: class and carry are compile-time, the lane enters as group 3 n
                ubo[0] = ubo[1] = (unsigned)(row0 + 3 * jc);
            } else {
                // (scale 2 and scale 4 alike: the pair's columns start 8 or 16 apart, two groups of SW columns)
                ubo[0] = (unsigned)(row0 + jx * NG + 2 * m);
                ubo[1] = (unsigned)(row0 + (jx ? 1 : (F::SW - 1) * NG) + 2 * m);
            }
        }
        const float* srow[F::RH0];                     // strip form: the lane half's filter rows in the ring
        if constexpr (STRIP != 0) {
#pragma unroll
            for (int dyv = 0; dyv < F::RH0; ++dyv) {
                const int s0 = slot0 + dyv, s1 = s0 + F::RH0;
                srow[dyv] = ring + (hf ? (s1 < F::SLOTS ? s1 : s1 - F::SLOTS) : (s0 < F::SLOTS ? s0 : s0 - F::SLOTS)) * (C * P) + jc;
            }
        }
        float outp[C][PX];
        float rinv[PX];                                // logits form: one over the sum of the pixel's exponentials
        if constexpr (LG) {
#pragma unroll
            for (int q = 0; q < PX; ++q) rinv[q] = __builtin_amdgcn_rcpf(acc[q][F::NSLOT / 16][F::NSLOT % 16]);   // the sum is at least 1
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if constexpr (PERM || PMAJ) {
                // The slots share few patch values (they are s pixels apart): taken all at once a channel's
                // LDS reads would hold three times the registers of the planar form.  One filter row at a
                // time; the empty statement ties the next row's addresses to this row's sums.
                static_assert(F::NSLOT % K == 0 && PX == 4, "whole filter rows per lane half");
                float sq[PX];
#pragma unroll
                for (int q = 0; q < PX; ++q) sq[q] = 0.0f;
#pragma unroll
                for (int dyv = 0; dyv < F::NSLOT / K; ++dyv) {
#pragma unroll
                    for (int q = 0; q < PX; ++q)
#pragma unroll
                        for (int dxv = 0; dxv < K; ++dxv) {
                            const int vv = dyv * K + dxv;
                            if constexpr (PMAJ) {
                                sq[q] = fmaf(acc[q][vv / 16][vv % 16], U[ubo[0] + c * UH * P + dyv * P + 32 * q + dxv], sq[q]);
                            } else if constexpr (PSM == 3) {
                                const int e = 3 * q + (unit % NSUB) + dxv;
                                sq[q] = fmaf(acc[q][vv / 16][vv % 16], U[ubo[0] + c * UH * P + dyv * P + (e & 3) * NG + (e >> 2)], sq[q]);
                            } else {
                                // column within the pair's group, before the lane's j is added; classes of SW columns
                                constexpr int SW = F::SW;
                                const int e0 = PSM == 4 ? 4 * q + 2 * (unit % NSUB) + dxv : 2 * q + dxv;
                                const bool wrap = e0 % SW == SW - 1;
                                const int imm = c * UH * P + dyv * P + (wrap ? 0 : (e0 % SW) * NG) + e0 / SW;
                                sq[q] = fmaf(acc[q][vv / 16][vv % 16], U[ubo[wrap ? 1 : 0] + imm], sq[q]);
                            }
                        }
                    asm volatile("" : "+v"(ubo[0]), "+v"(ubo[1]), "+v"(sq[0]), "+v"(sq[1]), "+v"(sq[2]), "+v"(sq[3]));
                }
#pragma unroll
                for (int q = 0; q < PX; ++q) outp[c][q] = LG ? sq[q] * rinv[q] : sq[q];
            } else {
#pragma unroll
                for (int q = 0; q < PX; ++q) {
                    float s = 0.0f;
#pragma unroll
                    for (int vv = 0; vv < F::NSLOT; ++vv) {
                        const int dyv = vv / K, dxv = vv % K;
                        if constexpr (STRIP != 0) {
                            s = fmaf(acc[q][vv / 16][vv % 16], srow[dyv][c * P + ((q + dxv) % PX) * NG + (q + dxv) / PX], s);
                        } else {
                            const int off = c * UH * P + dyv * P + ((q + dxv) % PX) * NG + (q + dxv) / PX;
                            s = fmaf(acc[q][vv / 16][vv % 16], ub[off], s);
                        }
                    }
                    outp[c][q] = LG ? s * rinv[q] : s;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }

        // (5) add the two halves' partial sums: one cross-half swap per slot pair
        //     leaves half 0 with pixels 0..PX/2-1 of the lane's group and half 1
        //     with the rest; one vector store per channel
        // (permuted slots: the lane's own pixels start at X0 + 4 PSM m; after the exchange below it stores
        //  the two adjacent pixels that start at X0 + 4 PSM m + 2 PSM hf + 2 (n % PSM))
        // (permuted slots, scale 4: the lane pair's pixels start at X0 + 16 m; a lane stores the four adjacent ones at
        //  X0 + 16 m + 8 hf + 4 j, once both units of the row are done)
        const int y = Y0 + unit_row(unit, wave) * WR + jr;
        // (scale 3: a lane's pixels start at X0 + 12 n; it stores the six adjacent ones at X0 + 12 n + 6 hf)
        // (pixel-major: half hf holds the lane's pixels 64 hf + j and 64 hf + 32 + j)
        const int x = PMAJ ? X0 + jc : PSM == 3 ? X0 + 12 * jc : (PERM ? X0 + 4 * PSM * (jc / 2) : X0 + PX * jc);
        const bool valid = y < a.H && x < a.W;
        const unsigned plane_px = (unsigned)a.H * (unsigned)a.W;
        const unsigned o0 = PMAJ ? (unsigned)y * (unsigned)a.W + x + hf * 64
                          : PSM == 3 ? (unsigned)y * (unsigned)a.W + x + hf * 6
                          : PERM ? (unsigned)y * (unsigned)a.W + x + hf * (2 * PSM) + (PSM == 4 ? 4 : 2) * (jc % 2)
                          : STRIP ? so0 : (unsigned)y * (unsigned)a.W + x + hf * (PX / 2);   // within the image
        char* const out_img = STRIP ? sout : (char*)a.out + (size_t)here.n * C * ((size_t)plane_px * (a.io_f16 ? 2 : 4));
        // Every lane stores, one outside the image at the end of the buffer, which drops it.  Behind a branch the compiler cannot
        // count the stores, and the next unit's fold, which waits for loads issued before them, waits for them as well.
        // 512 x 512 x4: 14.1 -> 13.3 us; no different where a unit is long.
        const unsigned out_bytes = C * plane_px * (a.io_f16 ? 2u : 4u);
        // (where no image can end in the last 64 bytes below 4 GB - scale 4, three channels at scale 3, lists and the forms with PSM >= 2, whose
        //  images are multiples of 64, 108, 96 and 192 bytes - a constant, which saves a scalar register: 1080p logits before the
        //  pixel-shuffle 80.4 -> 80.0 us)
        constexpr bool EVEN_END = LIST || PSM >= 2 || SMIN == 4 || (SMIN == 3 && C == 3);
        const unsigned beyond = EVEN_END ? 0xffffffc0u : out_bytes;
        const __amdgpu_buffer_rsrc_t out_rsrc = __builtin_amdgcn_make_buffer_rsrc(out_img, 0, (int)out_bytes, RAW_BUFFER);
#ifdef SR_ABLATE_STORES
        auto out_at = [&](unsigned e, unsigned size) -> unsigned { return valid && a.N < 0 ? e * size : beyond; };   // (never true)
#else
        auto out_at = [&](unsigned e, unsigned size) -> unsigned { return valid ? e * size : beyond; };
#endif
#pragma unroll
        for (int c = 0; c < C; ++c) {
            float tot[PX / 2];
            float tot4[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // scale-4 permuted slots: the four adjacent pixels a lane stores
            float tot6[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};   // scale 3: the six
#pragma unroll
            for (int q = 0; q < PX / 2; ++q) {
                const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(outp[c][q]),
                                                                 __float_as_uint(outp[c][q + PX / 2]), false, false);
                tot[q] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
            }
            if constexpr (PSM == 4) {
                // The lane pair (j = 0, 1) holds, per unit J, the pixels 16 m + 8 hf + {4 t + 2 J + j}, t = slot.
                // Unit J = 0 parks its two results; after unit J = 1 lane j' takes slot t = j' of both lanes and
                // both units: the four adjacent pixels 4 j' + {0, 1 | 2, 3} = {J = 0: j = 0, 1 | J = 1: j = 0, 1}.
                if (unit % NSUB == 0) {
                    park[c][0][0] = tot[0];
                    park[c][0][1] = tot[1];
                    continue;
                }
                const bool odd = (jc & 1) != 0;
                const unsigned g0 = __float_as_uint(odd ? park[c][0][0] : park[c][0][1]);    // what the partner stores
                const unsigned g1 = __float_as_uint(odd ? tot[0] : tot[1]);
                const float r0 = __uint_as_float(__builtin_amdgcn_update_dpp(0u, g0, 0xB1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
                const float r1 = __uint_as_float(__builtin_amdgcn_update_dpp(0u, g1, 0xB1, 0xf, 0xf, false));
                tot4[0] = odd ? r0 : park[c][0][0];
                tot4[1] = odd ? park[c][0][1] : r0;
                tot4[2] = odd ? r1 : tot[0];
                tot4[3] = odd ? tot[1] : r1;
            } else if constexpr (PSM == 3) {
                // Slot t of unit J is pixel 6 hf + 3 t + J of the lane's twelve: after the third unit the lane holds
                // the six adjacent ones (t = 0: J = 0, 1, 2; t = 1: J = 0, 1, 2).
                if (unit % NSUB != NSUB - 1) {
                    park[c][unit % NSUB][0] = tot[0];
                    park[c][unit % NSUB][1] = tot[1];
                    continue;
                }
                tot6[0] = park[c][0][0]; tot6[1] = park[c][1][0]; tot6[2] = tot[0];
                tot6[3] = park[c][0][1]; tot6[4] = park[c][1][1]; tot6[5] = tot[1];
            } else if constexpr (PSM == 2) {
                // The lane pair (j = 0, 1) holds the 4 pixels 8 m + 4 hf + {2 t + j}: lane j' takes 2 j', 2 j' + 1,
                // i.e. slot j' of both lanes of the pair.
                const unsigned t0 = __float_as_uint(tot[0]), t1 = __float_as_uint(tot[1]);
                const unsigned a0 = __builtin_amdgcn_update_dpp(0u, t0, 0xA0, 0xf, 0xf, false);   // quad_perm [0,0,2,2]
                const unsigned a1 = __builtin_amdgcn_update_dpp(0u, t1, 0xA0, 0xf, 0xf, false);
                const unsigned b0 = __builtin_amdgcn_update_dpp(0u, t0, 0xF5, 0xf, 0xf, false);   // quad_perm [1,1,3,3]
                const unsigned b1 = __builtin_amdgcn_update_dpp(0u, t1, 0xF5, 0xf, 0xf, false);
                const bool hi_slot = (jc & 1) != 0;
                tot[0] = __uint_as_float(hi_slot ? a1 : a0);
                tot[1] = __uint_as_float(hi_slot ? b1 : b0);
            }
            const unsigned oe = o0 + c * plane_px;
            if constexpr (PMAJ) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    if (a.io_f16) store16(out_rsrc, out_at(oe + 32 * t, 2u), tot[t]);
                    else store32(out_rsrc, out_at(oe + 32 * t, 4u), __float_as_uint(tot[t]));
                }
            } else if constexpr (PSM == 4) {
                if (a.io_f16) {
                    store64(out_rsrc, out_at(oe, 2u), pack_f16(tot4[0], tot4[1]), pack_f16(tot4[2], tot4[3]));
                } else {
                    store128(out_rsrc, out_at(oe, 4u), tot4);
                }
            } else if constexpr (PSM == 3) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    if (a.io_f16) store32(out_rsrc, out_at(oe + 2 * i, 2u), pack_f16(tot6[2 * i], tot6[2 * i + 1]));
                    else store64(out_rsrc, out_at(oe + 2 * i, 4u), __float_as_uint(tot6[2 * i]), __float_as_uint(tot6[2 * i + 1]));
                }
            } else if constexpr (PX == 4) {
                if (a.io_f16) store32(out_rsrc, out_at(oe, 2u), pack_f16(tot[0], tot[1]));
                else store_fp32_pair(out_rsrc, out_at(oe, 4u), tot[0], tot[1]);
            } else {
                static_assert(PX == 2, "two or four pixels per lane");
                if (a.io_f16) store16(out_rsrc, out_at(oe, 2u), tot[0]);
                else store32(out_rsrc, out_at(oe, 4u), __float_as_uint(tot[0]));
            }
        }
        // (6) L2 write-back pacing, see the note at the top of this file: workgroups 0 .. 7 run on the eight XCDs (fewer on a partition)
        if (a.wb_ticks > 0 && (int)blockIdx.x < a.wb_flushers && wave == 0) {
            const unsigned long long now = __builtin_amdgcn_s_memrealtime();
            if (now - wb_last >= (unsigned long long)a.wb_ticks) {
                wb_last = now;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            }
        }
    };
    if constexpr (STRIP != 0) {
        if constexpr (PTREG) {
#pragma unroll
            for (int i = 0; i < F::NLOAD; ++i) preg[i] = ptab[((tid0 >> 5) & 1) * F::NLOAD + i];
        }
        const unsigned esz = LIST ? 1u : OU;            // units of the coefficients' offsets: bytes (lists: elements)
        const size_t image_px = (size_t)a.H * a.W;
        auto lane_pix = [&](const TilePos p, int jc) -> unsigned {              // of a strip's row
            const int x = tile_x0(p.tx) + PX * jc, xc = x < a.W ? x : a.W - PX;
            return ((unsigned)p.ty * (unsigned)a.W + (unsigned)xc) * esz;
        };
        // the row whose coefficients are requested next: place of a segment's row
        auto ld_place = [&](const TilePos p, int jc) {
            spix = lane_pix(p, jc);
            snext = (const char*)a.coeff + (size_t)p.n * a.L * (image_px * F::CB);
            slist = (size_t)p.n * a.T * image_px;
        };
        ld_place(cur, tid0 & 31);
        const bool io_f16 = a.io_f16 != 0;
        for (int t = t_first; t < t_end; t += G) {
            int tid = tid0;
            asm volatile("" : "+v"(tid));
            const int lane = tid & 63, hf = lane >> 5, jc = lane & 31;
            TilePos sg = cur;                           // image, first row of the segment, strip
            if (t != t_first) {
                sg = tile_of(t);
                sg.ty *= a.seg_rows;
                strip_begin(sg, lane, io_f16);
            }
            const int y1 = min(a.H, sg.ty + a.seg_rows);
            strip_fence();
#pragma unroll
            for (int i = 0; i < 4; ++i) strip_store(sfloor - 1 + i, sinit[i], lane, io_f16);
            for (int i = -1; i < K; ++i) strip_rows(sg.ty - F::R + i, i, sg, lane, io_f16);
#pragma unroll
            for (int i = 0; i < LIT; ++i) asm volatile("" : "+v"(spre[i]));    // (there before the loop, or every round of it waits for everything)
            int slot = 0;                               // of row y - R
            so0 = (unsigned)sg.ty * (unsigned)a.W + (unsigned)(tile_x0(sg.tx) + PX * jc) + hf * (PX / 2);
            sout = (char*)a.out + (size_t)sg.n * C * (image_px * (io_f16 ? 2 : 4));
            auto step = [&](int parity, int y, const auto more) __attribute__((always_inline)) {
                strip_rows(y + F::R + 1, slot == 0 ? F::SLOTS - 1 : slot - 1, sg, lane, io_f16);
                strip_fence();
                int tid_row = tid;                      // (as `tid`: what a unit derives from it is not kept in registers across rows)
                asm volatile("" : "+v"(tid_row));
                const TilePos at = {sg.n, y, sg.tx};
                do_unit(parity, at, at, more, tid_row, slot, io_f16);
                so0 += (unsigned)a.W;
                slot = slot == F::SLOTS - 1 ? 0 : slot + 1;
            };
            auto inner = [&](int parity, int y) __attribute__((always_inline)) {     // a row with another after it in the segment
                spix += (unsigned)a.W * esz;
                step(parity, y, std::true_type{});
            };
            const bool more = t + G < t_end;
            auto before_last = [&]() {                  // what is requested next is the next segment's first row
                if (!more) return;
                TilePos sn = tile_of(t + G);
                sn.ty *= a.seg_rows;
                ld_place(sn, jc);
            };
            int y = sg.ty;
            if constexpr (LIST) {                       // two register sets
                for (; y + 2 < y1; y += 2) {
                    inner(0, y);
                    inner(1, y + 1);
                }
                if (y + 1 < y1) {
                    inner(0, y++);
                    before_last();
                    step(1, y, more);
                } else {
                    before_last();
                    step(0, y, more);
#pragma unroll
                    for (int e = 0; e < LH; ++e) { lval[0][e] = lval[1][e]; lidx[0][e] = lidx[1][e]; }
                }
            } else {
                for (; y + 1 < y1; ++y) inner(0, y);
                before_last();
                step(0, y, more);
            }
        }
    } else {
    for (int t = t_first; t < t_end; t += G) {
        // Per-iteration copy of the thread id the optimiser cannot see through:
        // index arithmetic derived from it is recomputed each tile instead of
        // being hoisted out of the loop into dozens of long-lived registers.
        int tid = tid0;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        const bool more_tiles = t + G < t_end;
        const TilePos nxt = more_tiles ? advance(cur) : cur;

        // (1) stage 1 of this tile.  (Spreading steps (a) and (b) of the next tile
        //     over the unit loop was measured slower: the extra mid-tile barrier and
        //     LDS traffic cost more than the shorter gap between tiles gains.)
        stage1_setup(cur, tid);
        __syncthreads();
#ifdef SR_ABLATE_STAGE1
        if (a.N < 0)
#endif
        stage1_vertical(cur, tid);
        __syncthreads();      // also: every wavefront is done with the previous tile's U
#ifdef SR_ABLATE_STAGE1
        if (a.N < 0)
#endif
        stage1_horizontal(tid);
        __syncthreads();
        // The wavefront's NU units of this tile, one after the other; while a unit
        // is folded, the coefficients of the next one (same tile, or unit 0 of the
        // next tile) are loaded into the registers that fall free.
#pragma unroll
        for (int unit = 0; unit < NU; ++unit) {
        do_unit(unit, cur, nxt, more_tiles, tid, 0, a.io_f16);
        // (2) prefetch the next tile's LR footprint from inside the unit loop, where
        //     the wavefront waits on memory anyway, and not in the barrier-to-barrier
        //     up-sampling phase that every wavefront of the workgroup has to sit out
        if (unit == (NU > 1 ? 1 : 0) && more_tiles) load_lr(nxt, lane, lrv, lrpar);
        }   // unit
        cur = nxt;
    }
    }
}

// rate of the constant clock s_memrealtime reads, in kHz (asked once per device and thread; 100 MHz if the runtime
// does not say)
inline long long wall_clock_khz() {
    static thread_local int known[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 100000;
    if (known[dev] == 0) {
        int khz = 0;
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz < 1000) khz = 100000;
        known[dev] = khz;
    }
    return known[dev];
}

// How `blocks` workgroups walk the tiles: each of 8 shares (the XCDs; one share if the grid is no multiple of 8) is a
// contiguous run of tiles, walked by every workgroup of that XCD in steps of their number.
inline void walk_of(AssembleArgs& a, int ntiles, int blocks, int per_block) {
    a.ntiles = ntiles;
    a.per_img = a.tiles_x * a.tiles_y;
    a.group_shift = blocks % 8 == 0 ? 3 : 0;
    const int groups = 1 << a.group_shift;
    a.share = (int)(((long long)ntiles + groups - 1) / groups);
    a.stride = blocks / groups * per_block;
    a.step_n = a.stride / a.per_img;
    const int r = a.stride - a.step_n * a.per_img;
    a.step_y = r / a.tiles_x;
    a.step_x = r - a.step_y * a.tiles_x;
    a.inv_img = (unsigned)((1ull << 32) / (unsigned)a.per_img - (a.per_img == 1 ? 1 : 0));
    a.inv_tx = (unsigned)((1ull << 32) / (unsigned)a.tiles_x - (a.tiles_x == 1 ? 1 : 0));
}

// Whether a call's coefficients are loaded with ordinary instead of streaming loads: rows that are no whole number of 128-byte lines, so that neighbouring tiles or
// strips share lines, which come from memory twice where the first reader lets them go (and streaming is 3 to 17 % faster where
// nothing is shared: 4K x4 fp16 244 / 278 us).  From frames of 400 thousand pixels on; smaller ones lie in the memory-side cache (0.95 to 1.04 of each other).
// 400 drawn calls, three states in turn, the same bits in all; streaming / ordinary us, and the ratios over the calls from the line on:
//   7x7: 2574 thousand pixels x3 121 atoms 200 / 158, 3308 thousand 72 atoms 1.23; all 1.00 .. 1.26, but one channel in rows off 128 bytes by 64 0.96 .. 1.07 (left)
//   5x5, 8-bit: 3175 thousand x3 78.5 / 66, 5391 thousand x1 119 / 99; 0.97 .. 1.25, mean 1.11, but by 64 0.96 .. 1.06 (left)
//   5x5, 16-bit, three channels: rows off 32 bytes 8035 thousand 46 atoms 245 / 191, 8306 thousand 316 / 290, 0.98 .. 1.28; rows off 128 only, which share
//   fewer lines: up to 40 atoms (less stream beside it) 1.02 .. 1.13, up to 72 0.94 .. 1.03 (left streaming), more from 2 million pixels 1.03 .. 1.12
//   (0.98 .. 1.00 below)
//   ... one channel: up to 50 atoms in rows off 32 bytes 1.00 .. 1.14; more 0.91 .. 1.04 (left streaming)
//   logits: rows off 64 bytes, and those off 32 with them, 1.00 .. 1.10; 64 of 128 bytes 0.96 (left)
//   3x3, three channels, 16- and 8-bit, from 1 million pixels: 1.10 .. 1.22
//   before the pixel-shuffle (rows of the LR image), values and logits (25 of 130 more calls): 5559 thousand x2 258 / 219, 5362 thousand x4 logits 232 / 198; 0.98 ..
//   1.18, by 64 bytes 0.94 .. 1.01 (left), whole lines 0.90 .. 1.02
// fp32: no gain was measured, not built.
inline bool keep_lines(const AssembleArgs& a, int k, bool logits) {
    const long long px = (long long)a.N * a.H * a.W;
    const bool f8 = a.coeff_dtype == SR_F8E4M3;
    const long long off = (long long)(a.pre_shuffle ? a.w : a.W) * (f8 ? 1 : 2) % 128;
    if (off == 0 || px < 400000) return false;
    if (logits || a.pre_shuffle) return off != 64;
    if (k == 7) return a.C == 3 || off != 64;
    if (k == 5 && f8) return off != 64;
    if (k == 3) return a.C == 3 && px >= 1000000;
    if (a.C == 1) return a.n_fold <= 50 && off % 32 != 0;
    if (a.C != 3) return false;
    return a.n_fold <= 40 || (a.n_fold <= 72 ? off % 32 != 0 : px >= 2000000);
}

template <int K, int C, int NP8, int PX, int WR, int NW, int NU, int WPE, int CT = CT_F16, int SMIN = 2, bool BIG = false,
          int PSM = 0, int STRIP = 0>
hipError_t launch_one(const AssembleArgs& a0, const LaunchTo& st) {
    using F = Cfg<K, C, NP8, PX, WR, NW, NU, CT, SMIN, (PSM == 4 ? 2 : (PSM == 3 ? 3 : 1)), (PSM == 8 ? 1 : 0), STRIP>;
    if (STRIP && a0.s != STRIP) return hipErrorInvalidValue;
    if (a0.s < SMIN) return hipErrorInvalidValue;       // its LDS footprint buffers would be too small
    if ((a0.pre_shuffle != 0) != (PSM >= 1 && PSM <= 4) || (a0.pixel_major != 0) != (PSM == 8)) return hipErrorInvalidValue;
    // logits: a softmax over every atom, so every plane is folded
    if ((a0.logits != 0) != (CT == CT_LOGIT || CT == CT_LOGIT_BF16) || (a0.logits && a0.n_fold != a0.L)) return hipErrorInvalidValue;
    if (a0.logits && (a0.coeff_dtype == SR_BF16) != (CT == CT_LOGIT_BF16)) return hipErrorInvalidValue;
    if (PSM == 8 && (a0.W % 128 != 0 || a0.L != 8 * NP8 || a0.n_fold != a0.L)) return hipErrorInvalidValue;
    if ((a0.blocked != 0) != (PSM == 9)) return hipErrorInvalidValue;
    if (PSM == 9 && (a0.W % 128 != 0 || a0.L != 8 * NP8 || a0.n_fold != a0.L)) return hipErrorInvalidValue;
    // permuted pixel slots: a lane owns four whole LR columns, the image must end on such a group
    if ((PSM == 2 || PSM == 3 || PSM == 4) && (a0.s != PSM || a0.w % 4 != 0)) return hipErrorInvalidValue;
    const int tiles_x = (a0.W + F::TW - 1) / F::TW;
    int tiles_y = (a0.H + F::TH - 1) / F::TH, xlast = (tiles_x - 1) * F::TW, seg_rows = F::TH;
    if (a0.W % PX != 0) {                               // ragged rows: the last tile column ends at the image edge
        if (a0.W < F::TW) return hipErrorInvalidValue;
        xlast = a0.W - F::TW;
        if (STRIP && xlast > 0 && xlast < F::R) return hipErrorInvalidValue;   // would look over the left edge, see strip_form
    }
    const int cap = units_of(a0) * (4 * WPE / NW > 0 ? 4 * WPE / NW : 1);
    if (STRIP) {
        // as many segments as there are wavefronts, or one per strip
        const long long strips = (long long)tiles_x * a0.N, waves = (long long)cap * NW;
        const int per_strip = (int)(strips < waves ? waves / strips : 1);
        seg_rows = (a0.H + per_strip - 1) / per_strip;
        tiles_y = (a0.H + seg_rows - 1) / seg_rows;
    }
    const long long nt = (long long)tiles_x * tiles_y * a0.N;
    if (nt > 0x7fffffffLL) return hipErrorInvalidValue;
    // as many workgroups as stay resident (WPE wavefronts per SIMD); strip form: a segment per wavefront
    const long long want = STRIP ? (nt + NW - 1) / NW : nt;
    const int blocks = want < cap ? (int)want : cap;
    if (st.walk) {
        *st.walk = {STRIP ? 2 : 1, F::TW, seg_rows, (int)nt, blocks, NW};
        return hipSuccess;
    }
    AssembleArgs a = a0;
#ifndef SR_NO_L2_WRITEBACK
    // L2 write-back pacing where the coefficient stream is the bound: 49 atoms and more, not the list forms nor 8-bit
    // coefficients in tiles (measured neutral at 43 kept atoms, 1-2 % slower below and for 8-bit tiles).  In strips 8-bit
    // coefficients are near the stream too: 4K 149.9 -> 146.4 us, 1080p x3 the same; strips with 8 atoms 60.8 -> 64.5 and lists
    // of 8 108 -> 111.5 with it, 4K fp16 strips 258 -> 245.
    if (NP8 >= 9 && (CT != CT_F8 || STRIP) && !F::LIST) {
        // 16 us of the constant-rate clock the kernel reads (7x7 atoms: 28 us, measured); one asking workgroup per XCD
        // (32 CUs each: eight on the whole device, fewer on a partition of it)
        a.wb_ticks = (int)((K == 7 ? 28LL : 16LL) * wall_clock_khz() / 1000);
        const int xcds = units_of(a0) / 32;
        a.wb_flushers = xcds < 1 ? 1 : (xcds > 8 ? 8 : xcds);
    }
#endif
    a.tiles_x = tiles_x;
    a.tiles_y = tiles_y;
    a.xlast = xlast;
    a.seg_rows = seg_rows;
    walk_of(a, (int)nt, blocks, STRIP ? NW : 1);
    constexpr bool LG = CT == CT_LOGIT || CT == CT_LOGIT_BF16;
    if constexpr ((PSM == 0 || PSM == 2 || PSM == 3 || PSM == 4) && !BIG && NP8 >= 4 && (C == 3 || (C == 1 && K != 3)) && (LG || CT == CT_F16 || CT == CT_BF16 || CT == CT_F8))
        if (keep_lines(a0, K, LG)) {
            hipLaunchKernelGGL((k_assemble_mfma<K, C, NP8, PX, WR, NW, NU, WPE, CT, SMIN, BIG, PSM, STRIP, true>), dim3(blocks), dim3(F::NT), 0, st.stream, a);
            return hipGetLastError();
        }
    hipLaunchKernelGGL((k_assemble_mfma<K, C, NP8, PX, WR, NW, NU, WPE, CT, SMIN, BIG, PSM, STRIP>), dim3(blocks), dim3(F::NT), 0, st.stream, a);
    return hipGetLastError();
}

// Whether a call goes to the strip form (strips of `sw` columns) where it is built next to tiles of tw x th pixels in
// workgroups of four wavefronts: the form that leaves the fullest SIMD with fewer rows; at about the same number the strips,
// which up-sample no row twice, once a segment is long enough to pay for its own first rows (scale 3: dearer rows).
// One column more than a strip is left to the tiles: its last strip would start at column 1 and see column -1, which the kernel
// continues for strips that start at column 0 only (continuing it there for all cost the light forms 1 % at every size).
// np8: capacity of the instantiation in groups of 8 atoms, 0 where the coefficient stream is not the bound (lists; fp32 with
// 7x7 atoms).
// Two cases in which strips are refused although the rows speak for them:
//   Rows that start on no multiple of 64 bytes, where the stream is the bound: instantiations for 48 atoms and more (one
//   channel: 32) filled to 97 % (90 %), more coefficients than the 256 MB memory-side cache can hold beside the rest (one
//   channel, which has half the other work to hide a miss behind: half of it), and work for 94 % of the resident lanes (128 atoms: 85 %).
//   Neighbouring pieces of a row then share lines.  Tiles side by side ask for them at about the same time; wavefronts that
//   walk strips drift apart, the loads are streaming ones, and the line comes from memory twice (with loads that stay in the
//   L2, 128 atoms 1536 x 2040 x3 263 -> 215 us, but whole lines 4K 239 -> 278: keep_lines, since when both forms take the same time there,
//   110 drawn calls within 2 %).  Strips have to save 8 % of the rows.
//   Scale 3, tiles of at most two rows per SIMD: a segment of one row up-samples K + 1 rows for it, one after the other; and
//   the same with up to three rows where a row is cheap to fold (one channel, few atoms, two pixels per lane) and strips save
//   at most a quarter of them.
// Measured, both forms in one run (us, tiles / strips; profiles/strips_or_tiles.txt has them and more):
//   fewer rows: 720p fp8 x4 34.2 / 24.8, 540 x 960 x2 fp16 29.1 / 23.9, 480 x 640 x2 fp32 33.3 / 28.5, 1080p x4 fp16 70.5 /
//   63.2
//   about the same: 4K x4, 8 atoms 80.2 / 62.7, 1080p x2 fp16 66.4 / 65.5, 4K x3 fp16 246.1 / 244.2, but 1080p x3 fp16 64.7 /
//   67.2 (segments of 8 rows)
//   rows that share lines: 1536 x 2040 x2 fp16 119.4 / 132.6, x3 with 7x7 atoms and one channel 119.8 / 144.3, 4K less 24
//   columns x4 fp16 287.8 / 308.8;
//   not refused: 1200 x 1608 x4 85.2 / 71.5 (92 % of the lanes), 1536 x 2040 x4 with 30 atoms 62.0 / 62.1, 900 x 1600 x2 fp8
//   with 45 atoms 34.5 / 28.7
//   segments of one row: 8 atoms, 240 x 312 x3 9.1 / 10.5, but 144 x 192 x2 9.1 / 8.7; of three: one channel, fp32, 8 atoms,
//   444 x 714 x3 10.2 / 11.2
inline bool strip_form(const AssembleArgs& a, int np8, int sw, int tw, int th, int wpe = 2) {
    if ((long long)a.C * a.H * a.W == (1ll << 30) - 1) return true;         // see the stores
    if (a.W == sw + 1) return false;                    // the moved last strip would start at column 1 and look over the left edge with R = 2
    const long long simds = 4ll * units_of(a), strips = (long long)((a.W + sw - 1) / sw) * a.N;
    const long long per_strip = strips < simds * wpe ? simds * wpe / strips : 1;
    const long long rows = (a.H + per_strip - 1) / per_strip, segments = strips * ((a.H + rows - 1) / rows);
    const long long tiles = (long long)((a.W + tw - 1) / tw) * ((a.H + th - 1) / th) * a.N;
    const long long strip_rows = (segments + simds - 1) / simds * rows;
    const long long tile_rows = (4 * tiles + simds - 1) / simds * (tw * th / (4 * sw));
    const long long row_bytes = (long long)a.W * (a.coeff_dtype == SR_F32 ? 4 : a.coeff_dtype == SR_F8E4M3 ? 1 : 2);
    const bool stream = np8 >= (a.C == 1 ? 4 : 6) && 100 * a.n_fold >= (a.C == 1 ? 90 : 97) * 8 * np8 &&
                        row_bytes * a.H * a.N * a.n_fold >= (a.C == 1 ? 128000000ll : 230000000ll) &&
                        100 * segments * a.W >= (np8 == 16 ? 85 : 94) * simds * wpe * ((a.W + sw - 1) / sw * sw);
    if (row_bytes % 64 != 0 && stream && 100 * strip_rows > 92 * tile_rows) return false;
    if (a.s == 3 && rows == 1 && tile_rows <= 2) return false;
    if (a.s == 3 && a.C == 1 && np8 >= 1 && np8 <= 2 && sw == 64 && rows <= 3 && 4 * strip_rows >= 3 * tile_rows) return false;
    return strip_rows < tile_rows || (10 * strip_rows <= 11 * tile_rows && rows >= (a.s == 3 ? 16 : 6));
}

// The strip form: workgroups of four wavefronts, WPE of them per CU.
template <int K, int C, int NP8, int PX, int WPE, int CT = CT_F16, int PSM = 0>
hipError_t launch_strip(const AssembleArgs& a, const LaunchTo& st) {
    constexpr int WPE2 = WPE < 3 ? WPE : 2;             // (scales 2 and 3: the LR rows of twelve wavefronts do not fit the LDS)
    switch (a.s) {
    case 2:  return launch_one<K, C, NP8, PX, 1, 4, 1, WPE2, CT, 2, false, PSM, 2>(a, st);
    case 3:  return launch_one<K, C, NP8, PX, 1, 4, 1, WPE2, CT, 3, false, PSM, 3>(a, st);
    case 4:  return launch_one<K, C, NP8, PX, 1, 4, 1, WPE, CT, 4, false, PSM, 4>(a, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace srd
