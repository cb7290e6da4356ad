// Normal equations of up to 79 atoms (k_atom_gram_split), and what the kernels of include/sr_select.h share.
#pragma once
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/sr_select.h"

namespace gram {

typedef float f32x4 __attribute__((ext_vector_type(4)));

struct GramArgs {
    const float* up;
    const void* coeff;
    const float* dict;
    const float* target;
    double* ws;
    int N, C, H, W, L, stride, ny, nx;
    int n16, ntile;              // 16-column blocks covering L + 1 columns, blocks in the upper triangle
};

inline int column_blocks(int L) { return (L + 1 + 15) / 16; }
inline int upper_blocks(int n) { return n * (n + 1) / 2; }

struct e4m3 { unsigned char bits; };        // 8-bit E4M3 storage, widened exactly by the conversion instruction
__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(__half v) { return __half2float(v); }
__device__ __forceinline__ float widen(e4m3 v) { return __builtin_amdgcn_cvt_f32_fp8((int)v.bits, 0); }
struct bf16v { unsigned short bits; };      // bfloat16 storage: the upper half of a binary32
__device__ __forceinline__ float widen(bf16v v) { return __uint_as_float((unsigned)v.bits << 16); }
// a coefficient as stored (loaded as an integer, which a load widens by itself), and back
template <int BYTES> struct BitsOf;
template <> struct BitsOf<4> { typedef unsigned type; };
template <> struct BitsOf<2> { typedef unsigned short type; };
template <> struct BitsOf<1> { typedef unsigned char type; };
template <typename TC>
__device__ __forceinline__ TC from_bits(unsigned b) {
    if constexpr (sizeof(TC) == 4) return __builtin_bit_cast(TC, b);
    else if constexpr (sizeof(TC) == 2) return __builtin_bit_cast(TC, (unsigned short)b);
    else return __builtin_bit_cast(TC, (unsigned char)b);
}
// x times the coefficient in bits 8 AT .. of a word (fp16: the half is widened by the multiplication itself)
template <typename TC, int AT>
__device__ __forceinline__ float times_stored(unsigned word, float x) {
    if constexpr (std::is_same<TC, __half>::value) {
        float r;
        if constexpr (AT == 0) asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(word), "v"(x));
        else asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(word), "v"(x));
        return r;
    } else {
        return widen(from_bits<TC>(word >> (8 * AT))) * x;
    }
}
__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

constexpr int NTT = 512;         // at most eight wavefronts
constexpr int GRIDT = 256;       // at most one workgroup per CU

// block b of the upper triangle of an N x N block matrix, row-major
template <int N>
struct UpperBlocks {
    int row[N * (N + 1) / 2], col[N * (N + 1) / 2];
    constexpr UpperBlocks() : row(), col() {
        int b = 0;
        for (int i = 0; i < N; ++i)
            for (int j = i; j < N; ++j) { row[b] = i; col[b] = j; ++b; }
    }
};

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// two floats as fp16, nearest even
__device__ __forceinline__ unsigned pack_halves(float x, float y) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    const f2 v = {x, y};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, h2));
}
__device__ __forceinline__ unsigned wave_max(unsigned m) {
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xf, 0xf, false));       // neighbours, pairs, quads, halves of a row
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xf, 0xf, false));
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xf, 0xf, false));
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x140, 0xf, 0xf, false));
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x142, 0xa, 0xf, false));      // rows 1 and 3 from the row before, then
    m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x143, 0xc, 0xf, false));      // the upper half from lane 31: lane 63 has all
    return (unsigned)__builtin_amdgcn_readlane((int)m, 63);
}
// the largest of lanes c16, c16 + 16, c16 + 32 and c16 + 48 (no NaN)
__device__ __forceinline__ float over_taps(float m) {
    auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    m = __builtin_elementwise_maximum(__uint_as_float(s[0]), __uint_as_float(s[1]));
    s = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    return __builtin_elementwise_maximum(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
// binary32 magnitudes: the exponent of one, a power of two
__device__ __forceinline__ int exponent_of(unsigned bits) { return (int)(bits >> 23) - 127; }
__device__ __forceinline__ float power_of_two(int e) { return __uint_as_float((unsigned)((e < 100 ? e : 100) + 127) << 23); }
// (v + grid_of(x)) - grid_of(x) is v, |v| <= x, to the nearest multiple of 2^-10 times x's power of two: an fp16 number, exactly
__device__ __forceinline__ float grid_of(float x) { return __uint_as_float(__float_as_uint(x) & 0x7f800000u) * 12288.0f; }
constexpr float TOP = 32768.0f;  // operands stay below
constexpr unsigned TOP_BITS = 0x47000000u;

// ---------------------------------------------------------------------------
// Many samples: k_atom_gram_tri (sr_select.hip) with its two contractions on the fp16 matrix instructions, whose rate is eight times that
// of the fp32 ones and which leave the vector units free.  Same items, same layouts, same order of items; a value enters as two fp16 parts
// (the dictionary as three), 24 bits.
//
// What makes the sums as good as fp32 ones: v_mfma_f32_16x16x32_f16 aligns the eight products of a lane to the largest exponent among them and cuts off what lies
// 2^-24 below it, towards zero, and adds such sums to the accumulator with few bits more than its own (measured with chosen
// operands).  Plain two-part operands are therefore biased (1e-8 in the normal equations of a 1080p frame, where fp32 sums have 5e-10).  So the large
// parts lie on a grid: v + m - m with m = 1.5 x 2^13 x the power of two of the largest value (of an operand's eight; of a sample's taps, of an atom's
// taps) is v to 11 bits of that largest one, so products of large parts are whole multiples of one unit, below 2^22 of them: nothing is cut off.  The small
// part is the rest, as fp16, and products with small parts are 2^-11 of the others: they have accumulators of their own (what is cut off there is beyond
// 2^-35) and are added to the large sums in fp32.  Against 64 bits, k_atom_gram_tri / this: G 5.0e-10 / 5.1e-10, b 3.8e-10 / 2.6e-10, h^T h 6.0e-10 /
// 5.5e-10 (1920 x 1080 x3, 72 atoms of 5x5); 608 x 848 x3 3x3, stride 2, 1.8e-9 / 1.1e-9, 1.6e-9 / 8.5e-10; 400 x 600 x3 7x7 60 atoms 9.5e-9 / 1.3e-9.
//
// An item of 16 samples and one channel takes 20 matrix instructions for the responses (5 blocks x 4 products, 25 of 32 taps) and 30 for the triangle (15 blocks x 4
// products, half of a 32-sample step) where fp32 takes 35 + 60 of twice the time.  Bound now: the vector instructions (some 300 an item: the
// parts of responses 80, doubles 45, the parts of the patch 55, responses 40) at two wavefronts per SIMD, beside which a matrix instruction still
// costs 5 to 9 cycles of issue (measured).  64 samples and channels are one batch: the operands of both 32-sample steps stay in registers (80), each block's
// sums are formed at once and added to its doubles, so no accumulator lives on; 9 of 15 blocks' doubles are in LDS.  Before / now, with up-sampling and
// the last sum, us: 1920 x 1080 x3 fp16 72 atoms of 5x5 648 / 406, 1000 x 1200 x1 bfloat16 60 atoms 126 / 101, 400 x 600 x3 7x7 60 atoms 98 / 74.
// Tried and not kept: flushing every 32 samples (fewer registers, 10 to 20 % slower), loads that differ by the item (coefficients of one load or of four: what
// is in flight is waited for where both meet, hence NEXT), several tap orders.
//
// Scales: image, responses and target are brought near 2^13 by powers of two that a wavefront takes from its first values other than zero and lowers where values
// pass 2^15 (adjust); sums are exact multiples, so they are rescaled in place.  Values far below the scale keep 2^-24 of 2^-1 absolute.
// Infinities and NaN: an atom that has them in a pair of items is contracted in fp32 for these, beside the others, and an image or dictionary that has
// them makes its responses tap by tap in fp32, so both go where k_atom_gram_tri takes them.
// ---------------------------------------------------------------------------
// NEXT: every pixel is a sample, in rows of four or more: a lane's four samples are one load.
template <int K, typename TC, int N16, bool NEXT>
__global__ __launch_bounds__(NTT, 2) void k_atom_gram_split(const GramArgs a, unsigned long long items) {
    constexpr int KK = K * K, R = (K - 1) / 2, KS = K == 3 ? 3 : (K == 5 ? 7 : 14);   // KS: taps of a lane
    constexpr int NK = (KS + 7) / 8;                                  // 32-tap steps of the responses
    constexpr int NB = N16 * (N16 + 1) / 2;
    constexpr UpperBlocks<N16> ub;
    // Sums of a wavefront's triangle in double: the first BR blocks in registers, the others, which with the operands would
    // not fit there, in LDS (each lane its own words).
    constexpr int BL = N16 == 5 ? (K == 7 ? 8 : 9) : (N16 == 4 ? 5 : 0), BR = NB - BL;
    constexpr int MAXB = BL > BR ? BL : BR;
    __shared__ double part[8 * MAXB * 256];
    __shared__ uint4 Bd[3 * NK * N16 * 64];                           // dictionary operand: parts, steps, blocks, lanes
    __shared__ unsigned dict_max[8];

    const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const size_t plane = (size_t)a.H * a.W;
    const int nseg = (a.nx + 15) / 16;

    // this wavefront's items
    const int nwaves = blockDim.x >> 6, NTH = blockDim.x;
    const unsigned nw = gridDim.x * nwaves, w = blockIdx.x * nwaves + wave;
    unsigned long long first, per;
    if (items <= 0xffffffffull) {
        const unsigned p = (unsigned)items / nw, rem = (unsigned)items - p * nw;
        first = (unsigned long long)w * p + (w < rem ? w : rem);
        per = p + (w < rem ? 1 : 0);
    } else {
        const unsigned long long p = items / nw, rem = items - p * nw;
        first = w * p + (w < rem ? w : rem);
        per = p + (w < rem ? 1 : 0);
    }
    int c, seg, iy, n;
    {
        const unsigned ipr = (unsigned)nseg * (unsigned)a.C;          // items of a lattice row (at most 2^16 x 16)
        unsigned long long row;
        unsigned r;
        if (first <= 0xffffffffull) {
            row = (unsigned)first / ipr;
            r = (unsigned)first - (unsigned)row * ipr;
        } else {
            row = first / ipr;
            r = (unsigned)(first - row * ipr);
        }
        seg = (int)(r / (unsigned)a.C);
        c = (int)(r - (unsigned)seg * (unsigned)a.C);
        n = row <= 0xffffffffull ? (int)((unsigned)row / (unsigned)a.ny) : (int)(row / (unsigned)a.ny);
        iy = (int)(row - (unsigned long long)n * (unsigned)a.ny);
    }

    const bool holds_target = c16 == (a.L & 15);                      // column L is the target: this lane's, in block L / 16
    constexpr int tblk = N16 - 1;                                     // (N16 blocks hold L + 1 columns, one fewer do not)

    // Slot j of lane (c16, q): a tap of sample c16 (or none: -1).  The first K slots are filter row q; 5x5: then a tap of row 4,
    // the fifth of them at q = 0; 7x7: then row q + 4.
    auto tap_of = [](int q, int j) {
        if (K == 3) return q < 3 ? q * K + j : -1;
        if (j < K) return q * K + j;
        if (K == 5) return j == 5 ? 20 + q : (q == 0 ? 24 : -1);
        return q < 3 ? (q + 4) * K + j - K : -1;
    };
    // Where an item's operands lie, from the first of the k image rows and from the lattice row: bytes of the lane's first filter row and of the other
    // taps, elements of the lane's samples.  Samples past the end of the row are clamped into it and their responses zeroed.
    unsigned off0 = 0, off1 = 0, off2 = 0, soff[NEXT ? 1 : 4];
    size_t top = 0, lattice_row = 0;                                  // elements before these rows in their plane
    int x0 = 0, left = 0;                                             // the item's first sample; samples that exist, from the lane's first on
    bool inside = false, whole = false;                               // no tap is clamped to the row; no sample is past its end
    auto place = [&](int iy_, int seg_) {
        const int Y = iy_ * a.stride, xl = a.nx - 1, first_row = max(Y - R, 0);
        x0 = seg_ * 16;
        left = a.nx - (x0 + 4 * kq);
        whole = x0 + 15 <= xl;
        inside = x0 * a.stride >= R && min(x0 + 15, xl) * a.stride + R < a.W;
        top = (size_t)first_row * a.W;
        lattice_row = (size_t)Y * a.W;
        auto row = [&](int dy) { return (unsigned)(clampi(Y + dy - R, 0, a.H - 1) - first_row) * (unsigned)a.W; };
        const int X = inside ? min(x0 + c16, xl) * a.stride - R : 0;  // (else the column is added tap by tap)
        off0 = 4u * (row(K == 3 && kq == 3 ? 2 : kq) + (unsigned)X);
        if constexpr (K == 5) {
            off1 = 4u * (row(4) + (unsigned)(inside ? X + kq : 0));
            off2 = off1 + (inside && kq == 0 ? 16u : 0u);
        }
        if constexpr (K == 7) off1 = 4u * (row(kq < 3 ? kq + 4 : 6) + (unsigned)X);
        if constexpr (NEXT) {
            soff[0] = (unsigned)min(x0 + 4 * kq, a.nx - 4);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) soff[e] = (unsigned)(min(x0 + 4 * kq + e, xl) * a.stride);
        }
    };
    size_t item_plane = ((size_t)n * a.C + c) * plane;                // elements before the item's channel
    float av[KS], h[4];
    auto fetch = [&]() {                                              // an item's patch operands and targets
        const char* const up = (const char*)(a.up + item_plane + top);
        const char* const tg = (const char*)(a.target + item_plane + lattice_row);
        if (inside) {
            typedef float four __attribute__((ext_vector_type(4), aligned(4)));
            typedef float three __attribute__((ext_vector_type(3), aligned(4)));
            if constexpr (K == 3) {
                const three v = *(const three*)(up + off0);
                av[0] = v[0]; av[1] = v[1]; av[2] = v[2];
            } else {
                const four v = *(const four*)(up + off0);
                av[0] = v[0]; av[1] = v[1]; av[2] = v[2]; av[3] = v[3];
                if constexpr (K == 5) {
                    av[4] = *(const float*)(up + off0 + 16);
                    av[5] = *(const float*)(up + off1);
                    av[6] = *(const float*)(up + off2);
                } else {
                    const three u = *(const three*)(up + off0 + 16), z = *(const three*)(up + off1 + 16);
                    const four y = *(const four*)(up + off1);
                    av[4] = u[0]; av[5] = u[1]; av[6] = u[2];
                    av[KS - 7] = y[0]; av[KS - 6] = y[1]; av[KS - 5] = y[2]; av[KS - 4] = y[3];
                    av[KS - 3] = z[0]; av[KS - 2] = z[1]; av[KS - 1] = z[2];
                }
            }
        } else {
            const int Xc = min(x0 + c16, a.nx - 1) * a.stride - R;
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                const int dx = j < K ? j : (K == 5 ? (j == 5 ? kq : 4) : j - K);
                av[j] = *(const float*)(up + ((j < K ? off0 : off1) + 4u * (unsigned)clampi(Xc + dx, 0, a.W - 1)));
            }
        }
        if constexpr (NEXT) {
            typedef float four __attribute__((ext_vector_type(4), aligned(4)));
            const four v = *(const four*)(tg + 4u * soff[0]);
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = v[e];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = *(const float*)(tg + 4u * soff[e]);
        }
    };
    // The coefficients of the lane's atoms and samples as stored (NEXT: four in RW words).  Lanes past the last atom take its plane
    // (the last block may hold the target column only: its first plane is the last atom's then).
    typedef typename BitsOf<sizeof(TC)>::type Bits;
    constexpr int RW = NEXT ? (int)sizeof(TC) : 4;
    unsigned raw[N16][RW];
    size_t img_plane = (size_t)n * a.L * plane;                       // elements before the image's coefficients
    const int last_block = 16 * (N16 - 1) < a.L ? 16 * (N16 - 1) : a.L - 1;
    const size_t plane_off = c16 * plane, plane_off_last = (last_block + c16 < a.L ? c16 : a.L - 1 - last_block) * plane;
    auto fetch_phi = [&]() {
        const Bits* const img = (const Bits*)a.coeff + img_plane + lattice_row;
#pragma unroll
        for (int nb = 0; nb < N16; ++nb) {
            const Bits* const at = img + (nb == N16 - 1 ? last_block : 16 * nb) * plane + (nb == N16 - 1 ? plane_off_last : plane_off);
            if constexpr (!NEXT) {
#pragma unroll
                for (int e = 0; e < 4; ++e) raw[nb][e % RW] = at[soff[NEXT ? 0 : e]];
            } else if constexpr (sizeof(TC) == 1) {
                struct __attribute__((packed, aligned(1))) word { unsigned v; };
                raw[nb][0] = ((const word*)(at + soff[0]))->v;
            } else {
                typedef unsigned words __attribute__((ext_vector_type(RW), aligned(sizeof(TC))));
                const words v = *(const words*)(at + soff[0]);
#pragma unroll
                for (int i = 0; i < RW; ++i) raw[nb][i] = v[i];
            }
        }
    };
    // NEXT: past the end of a row the lane's four are its last ones: sample e is element e + d of them (or zeroed)
    auto shifted = [&](const float (&v)[4], float (&w)[4]) {
        const int d = 4 - left;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = d <= 0 ? v[e] : (d == 1 ? v[e < 3 ? e + 1 : 3] : (d == 2 ? v[e < 2 ? e + 2 : 3] : v[3]));
    };
    if (per) {
        place(iy, seg);
        fetch();
        fetch_phi();
    }

    // The dictionary in three fp16 parts, times a power of two that brings its largest entry to 2^14; the large parts on one grid for an atom.
    // Lane (c16, kq), step nk, block nb: the taps of slots 8 nk .. 8 nk + 7, of atom 16 nb + c16.
    constexpr int DIT = (N16 * 64 + 255) / 256;                       // (for workgroups of 256 threads and more)
    float dv[DIT][8 * NK];
    unsigned dmax = 0;
#pragma unroll
    for (int it = 0; it < DIT; ++it) {
        const int e = tid + it * NTH, l64 = e & 63, l = 16 * (e >> 6) + (l64 & 15);
#pragma unroll
        for (int j = 0; j < 8 * NK; ++j) {
            const int tap = j < KS ? tap_of(l64 >> 4, j) : -1;
            dv[it][j] = (e < N16 * 64 && l < a.L && tap >= 0) ? a.dict[l * KK + tap] : 0.0f;
        }
    }
#pragma unroll
    for (int it = 0; it < DIT; ++it)
#pragma unroll
        for (int j = 0; j < 8 * NK; ++j) dmax = max(dmax, __float_as_uint(dv[it][j]) & 0x7fffffffu);
    dmax = wave_max(dmax);
    if (lane == 0) dict_max[wave] = dmax;
    __syncthreads();
    for (int v = 0; v < nwaves; ++v) dmax = max(dmax, dict_max[v]);
    const bool dict_finite = dmax < 0x7f800000u;
    const float sD = dict_finite && dmax != 0 ? power_of_two(14 - exponent_of(dmax)) : 1.0f;
#pragma unroll
    for (int it = 0; it < DIT; ++it) {
        const int e = tid + it * NTH;
        float mx = 0.0f, p[3][8 * NK];
#pragma unroll
        for (int j = 0; j < 8 * NK; ++j) mx = __builtin_elementwise_maximum(mx, fabsf(dv[it][j] * sD));
        const float magic = grid_of(over_taps(mx));
#pragma unroll
        for (int j = 0; j < 8 * NK; ++j) {
            const float d = dv[it][j] * sD;
            p[0][j] = (d + magic) - magic;
            p[1][j] = (float)(_Float16)(d - p[0][j]);
            p[2][j] = (d - p[0][j]) - p[1][j];
        }
        if (e < N16 * 64) {
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
                for (int k = 0; k < NK; ++k)
                    Bd[(q * NK + k) * (N16 * 64) + e] = make_uint4(pack_halves(p[q][8 * k], p[q][8 * k + 1]), pack_halves(p[q][8 * k + 2], p[q][8 * k + 3]),
                                                                   pack_halves(p[q][8 * k + 4], p[q][8 * k + 5]), pack_halves(p[q][8 * k + 6], p[q][8 * k + 7]));
        }
    }

    double dacc[BR][4];
#pragma unroll
    for (int b = 0; b < BR; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) dacc[b][e] = 0.0;
    double* const mine = part + wave * (MAXB * 256) + lane;
#pragma unroll
    for (int i = 0; i < 4 * BL; ++i) mine[64 * i] = 0.0;
    __syncthreads();                                                  // the dictionary operand is written

    // Powers of two: of the image, of the responses and of the target (their operands are the values times these).  One of
    // them is set where the first values other than zero come, and lowered where values leave its range.
    float sB = 1.0f, sR = 1.0f, sT = 1.0f;
    bool setB = false, setR = false, setT = false;
    float phi[N16][4];                                                // coefficients times sR / (sB sD)
    const auto to_dots = [&]() { return sR / (sB * sD); };

    unsigned oh[2][N16][4], om[2][N16][4];                            // operands of 32 samples each: large parts, small parts
    auto half8_of = [](const unsigned (&v)[4]) { return __builtin_bit_cast(f16x8, u32x4{v[0], v[1], v[2], v[3]}); };
    auto add_block = [&](int b, const f32x4& v) {
        if (b < BR) {
#pragma unroll
            for (int e = 0; e < 4; ++e) dacc[b < BR ? b : 0][e] += (double)v[e];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) mine[64 * (4 * (b - BR) + e)] += (double)v[e];
        }
    };
    constexpr int G = 3;                                                       // blocks whose matrix instructions take turns
    // the triangle over 32 or 64 samples
    auto contract = [&](const auto both) __attribute__((always_inline)) {
        constexpr int ST = both.value ? 2 : 1;
#pragma unroll
        for (int b0 = 0; b0 < NB; b0 += G) {
            f32x4 large[G], small[G];
#pragma unroll
            for (int g = 0; g < G; ++g) large[g] = small[g] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            auto step = [&](f32x4 (&acc)[G], const auto& x, const auto& y) {
#pragma unroll
                for (int g = 0; g < G; ++g)
                    if (b0 + g < NB)
                        acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(half8_of(x[ub.row[b0 + g < NB ? b0 + g : 0]]), half8_of(y[ub.col[b0 + g < NB ? b0 + g : 0]]), acc[g], 0, 0, 0);
            };
#pragma unroll
            for (int s = 0; s < ST; ++s) {
                step(small, om[s], om[s]);
                step(small, om[s], oh[s]);
                step(large, oh[s], oh[s]);
                step(small, oh[s], om[s]);
            }
#pragma unroll
            for (int g = 0; g < G; ++g)
                if (b0 + g < NB) add_block(b0 + g, large[g] + small[g]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    f32x4 r0[N16], r1[N16];                                           // responses (and target) of two items
    // Rare: values without a scale yet, out of their scale's range, or not finite.
    auto adjust = [&](const auto half) __attribute__((always_inline)) {
        unsigned mr = 0, mt = 0, bad = 0;                             // bit nb: the atom of block nb and this lane has infinities or NaN
#pragma unroll
        for (int nb = 0; nb < N16; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned v = max(__float_as_uint(r0[nb][e]) & 0x7fffffffu, __float_as_uint(r1[nb][e]) & 0x7fffffffu);
                if (v >= 0x7f800000u) bad |= 1u << nb;
            }
        bad |= (unsigned)__shfl_xor((int)bad, 16);
        bad |= (unsigned)__shfl_xor((int)bad, 32);
#pragma unroll
        for (int nb = 0; nb < N16; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned v = max(__float_as_uint(r0[nb][e]) & 0x7fffffffu, __float_as_uint(r1[nb][e]) & 0x7fffffffu);
                if (bad >> nb & 1) continue;
                if (nb == tblk && holds_target) mt = v > mt ? v : mt;
                else mr = v > mr ? v : mr;
            }
        mr = wave_max(mr);
        mt = wave_max(mt);
        float fr = 1.0f, ft = 1.0f;
        if (mr != 0 && (!setR || mr >= TOP_BITS)) { fr = power_of_two(13 - exponent_of(mr)); setR = true; }
        if (mt != 0 && (!setT || mt >= TOP_BITS)) { ft = power_of_two(13 - exponent_of(mt)); setT = true; }
        if (fr != 1.0f || ft != 1.0f) {
            if constexpr (half.value == 1) {                          // (the first half's operands carry the old scale)
                contract(std::false_type{});
#pragma unroll
                for (int nb = 0; nb < N16; ++nb)
#pragma unroll
                    for (int i = 0; i < 4; ++i) oh[0][nb][i] = om[0][nb][i] = 0;
            }
            sR *= fr;
            sT *= ft;
#pragma unroll
            for (int nb = 0; nb < N16; ++nb) {
                const float f = nb == tblk && holds_target ? ft : fr;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    r0[nb][e] *= f;
                    r1[nb][e] *= f;
                    phi[nb][e] *= fr;
                }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double f = (double)(ub.col[b] == tblk && holds_target ? ft : fr) * (double)(ub.row[b] == tblk && 4 * kq + e == (a.L & 15) ? ft : fr);
                    if (b < BR) dacc[b < BR ? b : 0][e] *= f;
                    else mine[64 * (4 * (b - BR) + e)] *= f;
                }
        }
        if (__builtin_amdgcn_ballot_w64(bad != 0)) {                  // these atoms' products in fp32, as they come
            unsigned badr[4];                                         // of this lane's rows
#pragma unroll
            for (int e = 0; e < 4; ++e) badr[e] = (unsigned)__shfl((int)bad, 4 * kq + e);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(r0[ub.row[b]][e], r0[ub.col[b]][e], acc, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(r1[ub.row[b]][e], r1[ub.col[b]][e], acc, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = (bad >> ub.col[b] & 1) || (badr[e] >> ub.row[b] & 1) ? acc[e] : 0.0f;
                add_block(b, acc);
            }
#pragma unroll
            for (int nb = 0; nb < N16; ++nb)
                if (bad >> nb & 1) r0[nb] = r1[nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    };
    // two items' responses as operands
    auto convert = [&](const auto half) __attribute__((always_inline)) {
        constexpr int s = half.value;
        float m8[N16];                                                // (NaN stays)
        auto largest = [&]() {
#pragma unroll
            for (int nb = 0; nb < N16; ++nb) {
                m8[nb] = __builtin_elementwise_maximum(fabsf(r0[nb][0]), fabsf(r1[nb][0]));
#pragma unroll
                for (int e = 1; e < 4; ++e) m8[nb] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m8[nb], fabsf(r0[nb][e])), fabsf(r1[nb][e]));
            }
        };
        largest();
        float top = m8[0];
#pragma unroll
        for (int nb = 1; nb < N16; ++nb) top = __builtin_elementwise_maximum(top, m8[nb]);
        if (!setR || !setT || __builtin_amdgcn_ballot_w64(!(top < TOP)) != 0) {
            adjust(half);
            largest();
        }
#pragma unroll
        for (int nb = 0; nb < N16; ++nb) {
            const float magic = grid_of(m8[nb]);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const f32x4 v = i == 0 ? r0[nb] : r1[nb];
                float g[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] = (v[e] + magic) - magic;
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    oh[s][nb][2 * i + p] = pack_halves(g[2 * p], g[2 * p + 1]);
                    om[s][nb][2 * i + p] = pack_halves(v[2 * p] - g[2 * p], v[2 * p + 1] - g[2 * p + 1]);
                }
            }
        }
    };
    bool first_item = true;
    // an item's responses
    auto item = [&](f32x4 (&r)[N16]) __attribute__((always_inline)) {
        if (c == 0 || first_item) {                                   // 16 samples' coefficients
            first_item = false;
            const float f = to_dots();
#pragma unroll
            for (int nb = 0; nb < N16; ++nb) {
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = widen(from_bits<TC>(NEXT ? raw[nb][e * RW / 4] >> (8 * RW * e % 32) : raw[nb][e % RW]));
                if (NEXT && !whole) shifted(v, v);
#pragma unroll
                for (int e = 0; e < 4; ++e) phi[nb][e] = f * v[e];
            }
        }
        float b[KS], mb = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            b[ks] = (K == 3 && kq == 3) || (K == 5 && ks == 6 && kq != 0) || (K == 7 && ks >= K && kq == 3) ? 0.0f : av[ks];   // (no tap)
            mb = __builtin_elementwise_maximum(mb, fabsf(b[ks]));
        }
        bool in_fp32 = !dict_finite;
        if (!setB || __builtin_amdgcn_ballot_w64(!(mb * sB < TOP)) != 0) {      // rare, as in adjust
            const unsigned bits = __float_as_uint(mb) & 0x7fffffffu;
            const unsigned mx = wave_max(bits < 0x7f800000u ? bits : 0u);
            in_fp32 = in_fp32 || __builtin_amdgcn_ballot_w64(bits >= 0x7f800000u) != 0;
            if (mx != 0 && (!setB || !(__uint_as_float(mx) * sB < TOP))) {
                const float f = to_dots();
                sB = power_of_two(13 - exponent_of(mx));
                setB = true;
                const float by = to_dots() / f;
#pragma unroll
                for (int nb = 0; nb < N16; ++nb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) phi[nb][e] *= by;
            }
        }
        unsigned bh[NK][4], bm[NK][4];
        {
            const float magic = grid_of(over_taps(mb) * sB);            // one grid for a sample
            float g[8 * NK], m[8 * NK];
#pragma unroll
            for (int i = 0; i < 8 * NK; ++i) {
                const float v = i < KS ? b[i < KS ? i : 0] * sB : 0.0f;
                g[i] = i < KS ? (v + magic) - magic : 0.0f;
                m[i] = i < KS ? v - g[i] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < 4 * NK; ++i) {
                bh[i / 4][i % 4] = pack_halves(g[2 * i], g[2 * i + 1]);
                bm[i / 4][i % 4] = pack_halves(m[2 * i], m[2 * i + 1]);
            }
        }
        const int here = left;
        const bool all_here = whole;
        float ht[4] = {h[0], h[1], h[2], h[3]};
        if (NEXT && !whole) shifted(ht, ht);
        // the next item's patch operands and targets, and its coefficients where they are others (after the wavefront's last
        // item: the same again, unused)
        const bool last_channel = c + 1 == a.C;
        --per;
        if (per != 0) {
            if (last_channel) {
                c = 0;
                item_plane -= (a.C - 1) * plane;
                if (++seg == nseg) {
                    seg = 0;
                    if (++iy == a.ny) {
                        iy = 0;
                        item_plane += a.C * plane;
                        img_plane += a.L * plane;
                    }
                }
                place(iy, seg);
            } else {
                ++c;
                item_plane += plane;
            }
        }
        fetch();
        if (last_channel) fetch_phi();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b0 = 0; b0 < N16; b0 += G) {
            f32x4 large[G], small[G];
#pragma unroll
            for (int g = 0; g < G; ++g) large[g] = small[g] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            auto step = [&](f32x4 (&acc)[G], int part_, const auto& x) {
#pragma unroll
                for (int nk = 0; nk < NK; ++nk)
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        if (b0 + g < N16)
                            acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(half8_of(x[nk]), __builtin_bit_cast(f16x8, Bd[(part_ * NK + nk) * (N16 * 64) + (b0 + g) * 64 + lane]), acc[g], 0, 0, 0);
            };
            step(small, 2, bh);
            step(small, 1, bh);
            step(large, 0, bh);
            step(small, 0, bm);
#pragma unroll
            for (int g = 0; g < G; ++g)
                if (b0 + g < N16) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) r[b0 + g < N16 ? b0 + g : 0][e] = (large[g][e] + small[g][e]) * phi[b0 + g < N16 ? b0 + g : 0][e];
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (in_fp32) {                                                // infinities or NaN in the image or the dictionary: tap by tap
            const float s = sB * sD;
            f32x4 sum[N16];
#pragma unroll
            for (int nb = 0; nb < N16; ++nb) sum[nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll 1
                for (int q = 0; q < 4; ++q) {
                    const int tap = tap_of(q, ks);
                    if (tap < 0) continue;
                    float bt[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) bt[e] = __shfl(b[ks], 4 * kq + e + 16 * q);
#pragma unroll
                    for (int nb = 0; nb < N16; ++nb) {
                        const int l = 16 * nb + c16;
                        const float d = l < a.L ? a.dict[l * KK + tap] : 0.0f;
#pragma unroll
                        for (int e = 0; e < 4; ++e) sum[nb][e] = fmaf(bt[e], d, sum[nb][e]);
                    }
                }
#pragma unroll
            for (int nb = 0; nb < N16; ++nb)
#pragma unroll
                for (int e = 0; e < 4; ++e) r[nb][e] = sum[nb][e] * s * phi[nb][e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) r[tblk][e] = holds_target ? ht[e] * sT : r[tblk][e];
        if (!all_here) {                                              // the end of a row
#pragma unroll
            for (int nb = 0; nb < N16; ++nb)
#pragma unroll
                for (int e = 0; e < 4; ++e) r[nb][e] = e < here ? r[nb][e] : 0.0f;
        }
    };
    typedef std::integral_constant<int, 0> First;
    typedef std::integral_constant<int, 1> Second;
    auto none = [&](f32x4 (&r)[N16]) {
#pragma unroll
        for (int nb = 0; nb < N16; ++nb) r[nb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    };
    while (per != 0) {
        const int count = per < 4 ? (int)per : 4;
        item(r0);
        if (count > 1) item(r1); else none(r1);
        convert(First{});
        if (count > 2) {
            item(r0);
            if (count > 3) item(r1); else none(r1);
            convert(Second{});
            contract(std::true_type{});
        } else {
            contract(std::false_type{});
        }
    }
    {
        const double uR = 1.0 / (double)sR, uT = 1.0 / (double)sT;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const double u = (ub.col[b] == tblk && holds_target ? uT : uR) * (ub.row[b] == tblk && 4 * kq + e == (a.L & 15) ? uT : uR);
                if (b < BR) dacc[b < BR ? b : 0][e] *= u;
                else mine[64 * (4 * (b - BR) + e)] *= u;
            }
    }

    // The workgroup's sum, wavefront by wavefront: the blocks in LDS, then, in their place, those in registers.
    // Lane (c16, kq), register e of block (bi, bj) holds row 16 bi + 4 kq + e, column 16 bj + c16.
    auto add_up = [&](int first_block, int blocks) {
        __syncthreads();
        for (int i = tid; i < blocks * 256; i += NTH) {
            double sum = 0.0;
            for (int v = 0; v < nwaves; ++v) sum += part[v * (MAXB * 256) + i];
            a.ws[((size_t)blockIdx.x * NB + first_block) * 256 + (size_t)(i >> 8) * 256 + (i & 63) * 4 + ((i >> 6) & 3)] = sum;
        }
    };
    if constexpr (BL != 0) {
        add_up(BR, BL);
        __syncthreads();
    }
#pragma unroll
    for (int b = 0; b < BR; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) mine[64 * (4 * b + e)] = dacc[b][e];
    add_up(0, BR);
}

template <int K, typename TC, int N16>
static hipError_t launch_split_n(const GramArgs& a, unsigned long long items, int grid, hipStream_t st) {
    if (a.stride == 1 && a.nx >= 4) hipLaunchKernelGGL((k_atom_gram_split<K, TC, N16, true>), dim3(grid), dim3(NTT), 0, st, a, items);
    else hipLaunchKernelGGL((k_atom_gram_split<K, TC, N16, false>), dim3(grid), dim3(NTT), 0, st, a, items);
    return hipGetLastError();
}

template <int K, typename TC>
static hipError_t launch_split_t(const GramArgs& a, unsigned long long items, int grid, hipStream_t st) {
    if constexpr (K == 7)
        if (a.n16 == 2) return launch_split_n<K, TC, 2>(a, items, grid, st);
    if constexpr (K != 3) {
        if (a.n16 == 3) return launch_split_n<K, TC, 3>(a, items, grid, st);
        if (a.n16 == 4) return launch_split_n<K, TC, 4>(a, items, grid, st);
    }
    if constexpr (K != 7)
        if (a.n16 == 5) return launch_split_n<K, TC, 5>(a, items, grid, st);
    return hipErrorInvalidValue;
}

template <int K>
static hipError_t launch_split_k(const GramArgs& a, int coeff_dtype, unsigned long long items, int grid, hipStream_t st) {
    switch (coeff_dtype) {
    case SR_F16:  return launch_split_t<K, __half>(a, items, grid, st);
    case SR_F32:  return launch_split_t<K, float>(a, items, grid, st);
    case SR_BF16: return launch_split_t<K, bf16v>(a, items, grid, st);
    default:      return launch_split_t<K, e4m3>(a, items, grid, st);
    }
}

// Which calls k_atom_gram_split serves faster than k_atom_gram_tri: it starts later (the dictionary's parts, the scales, more code to fetch: 2 to
// 4 us) and gains with the number of blocks and items.  k_atom_gram_tri / this, us (378 drawn calls): 5x5, five blocks (64 to 79
// atoms) 3108 items 23 / 26, 5148 items 22.2 / 22.6, 6690 items 26.8 / 24.0, 13419 items 40 / 37, 55104 items 1.32 of each other, 388800 items
// 617 / 372; three blocks 4671 items 13.1 / 13.6, 8094 items 15.6 / 15.2, 50676 items 1.28; two blocks and one 0.83 to 1.13 at any size.
// 3x3, five blocks 5508 items 20 / 22, 13860 items 39 / 36, 53958 items 1.24; fewer blocks 0.84 to 1.06.  7x7, two to four blocks 6500
// items 1.03 to 1.15, 40000 items 1.13 to 1.4; one block 0.88 to 1.4; five do not fit the registers (0.54 to 1.12).  One channel, whose coefficients serve
// one item: 5x5, five blocks 10175 items 38.5 / 40.8, 15876 items 1.12; 3x3 fp32 32852 items 69 / 73.
inline bool split_faster(int k, int n16, int channels, int coeff_dtype, unsigned long long items) {
    if (k == 3 ? n16 != 5 || (channels == 1 && coeff_dtype == SR_F32) : k == 5 ? n16 < 3 : n16 < 2 || n16 > 4) return false;
    return items >= (channels == 1 ? 16384u : k == 5 && n16 == 5 ? 6144u : 8192u);
}

hipError_t launch_split_k3(const GramArgs& a, int coeff_dtype, unsigned long long items, int grid, hipStream_t st);
hipError_t launch_split_k5(const GramArgs& a, int coeff_dtype, unsigned long long items, int grid, hipStream_t st);
hipError_t launch_split_k7(const GramArgs& a, int coeff_dtype, unsigned long long items, int grid, hipStream_t st);

}  // namespace gram
