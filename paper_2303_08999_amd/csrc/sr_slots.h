// Matrix-core kernel for calls that the streaming kernel (sr_mfma_kernel.h) has no instantiation for: coefficients before the
// network's pixel-shuffle and logits, for every coefficient type, atom size and scale, one to three channels, up to 128 folded
// atoms, any width; planar coefficients in two channels, narrow ragged frames and the like; and calls of the streaming kernel, of either order, that are
// faster here (slots_faster).  All but the last ran on the generic kernel, which folds on the
// vector ALUs and reads a pixel's coefficients eight at a time, one memory latency after the other: that is what bounded all but the
// largest of them.  Here a wavefront takes a UNIT, 32 lanes times the pixels of a 32-bit word of coefficients, requests all of its
// coefficients at once, and folds it on the matrix cores.
//
// One instantiation serves every layout: what differs is where a unit's words lie.  In the planar order they are 32 P neighbouring
// pixels of a row (P = 4, 2 or 1 pixels in a word of 8-, 16- or 32-bit coefficients).  Before the pixel-shuffle they are 32 P
// neighbouring LR pixels of ONE sub-pixel plane, i.e. HR pixels s apart, so that a wavefront's load reads whole memory lines there too;
// the s units of a row are the s sub-pixel columns.  Either way lane j of a half holds the unit's pixels P j .. P j + P - 1 (its
// slots), the half's atoms as in sr_mfma_kernel.h, and slot q is tile column e + SW j with SW = s P (planar: P) and e = s q +
// sub-pixel column.  The up-sampled tile is stored by classes modulo SW, so that the lanes of a read have neighbouring words: column x
// at (x % SW) NG + x / SW.
//
// What bounds it now: for large frames of many atoms the coefficients (logits 1638 x 1608 x1, 128 atoms: 153 us, 4.5 TB/s), for three
// channels the filtering, whose slots share no patch values, and the up-sampling (together half of a 1020 x 1060 x3 frame), for small
// ones the latency of one tile.  Generic kernel / this one, us: before the pixel-shuffle, 216 x 230 x3 fp16 72 atoms 28 / 12, 1020 x
// 1060 x3 bfloat16 72 atoms 120 / 48, fp8 110 / 59, fp32 133 / 75; logits, 180 x 234 x1 fp16 72 atoms 46 / 13, 1104 x 687 x3 bfloat16 104
// atoms of 3x3 118 / 49, 1152 x 945 x3 fp16 128 atoms of 7x7 342 / 96.
//
// Precision: fp32 coefficients go through v_mfma_f32_32x32x2_f32 (products and sums fp32).  16- and 8-bit ones and the
// exponentials of logits meet the dictionary as 16-bit parts: fp16, of the dictionary scaled by one power of two, the first part and the
// rest times 2^11 into a sum of its own, 22 significant bits of every entry down to 2^-29 of the largest; bfloat16 three parts, 24 bits.
// (Calls of the streaming kernel: its parts, its order, its bits.)  Against 64-bit arithmetic two drawn calls went from
// 1.0e-7 and 1.1e-7 in the generic kernel to 7.6e-8 and 6.8e-8.
#pragma once
#include <string.h>

#include "sr_mfma_kernel.h"

namespace srd {

struct SlotArgs {
    const void*  lr;
    const void*  coeff;
    const float* dict;
    void*        out;
    int N, C, h, w, H, W, s, L, n_fold, io_f16, identity;
    int upr, th;                 // units of a tile row, rows of a tile
    int sw, ng;                  // column classes of the tile, stride between them
    unsigned inv_sw;             // ceil(2^16 / sw)
    int tiles_x, tiles_y, ntiles, share, stride, group_shift;      // (how they are dealt to the workgroups: as in AssembleArgs)
    int   kept[SR_MAX_ATOMS];
    float gamma[SR_MAX_ATOMS];
};

// What a call brings: coefficients or logits, whose dictionary keeps (nearly) all bits of fp32 as in the generic kernel, which served them
// before; or coefficients that the streaming kernel has an instantiation for too: its two parts in one sum, in its order, so that these calls have
// its bits, whichever kernel their size sends them to.
constexpr int SLOT_VALUES = 0, SLOT_LOGITS = 1, SLOT_STREAMED = 2;

template <int K, int CM, int CT, int NP8, int KIND, bool PRE>
struct SlotCfg {
    static constexpr bool LG = KIND == SLOT_LOGITS, ST = KIND == SLOT_STREAMED;
    static constexpr int KK = K * K, R = (K - 1) / 2, RH0 = (K + 1) / 2, NSLOT = RH0 * K, NMB = (NSLOT + 15) / 16;
    static constexpr int CB = CT == CT_F32 ? 4 : (CT == CT_F8 ? 1 : 2), P = 4 / CB;      // bytes of a coefficient, pixels of a word
    static constexpr bool F32 = CT == CT_F32 && !LG;                   // fp32 matrix instructions
    static constexpr bool BF = CT == CT_BF16 && !LG;                   // bfloat16 ones (logits: fp16, whatever they are stored as)
    static constexpr int NPART = F32 ? 1 : (BF && !ST ? 3 : 2);        // 16-bit parts of a dictionary entry
    static constexpr int NACC = F32 || BF || ST ? 1 : 2;               // sums: fp16's second part has its own
    // fp16 parts: of the dictionary times a power of two that brings its largest entry below 2^15.  Unscaled, entries of 65520 and more overflow and
    // small ones keep 2^-35 at best.
    static constexpr bool SCALED = NACC == 2;
    static constexpr int QG = P * NMB * NACC <= 4 ? P : (NMB * NACC <= 2 ? 2 : 1);   // slots folded together (registers)
    static constexpr int QGP = QG < P ? QG : P;
    static constexpr int N16 = F32 ? 0 : NP8 / 2, N8 = F32 ? 0 : NP8 % 2, N2 = F32 ? 4 * NP8 : 0;
    static constexpr int NLOAD = 4 * NP8;
    // Most rows of a tile (a large frame up-samples the fewer rows twice the taller its tiles are), and wavefronts per SIMD: the
    // filtering waits for LDS and hides behind other wavefronts, so three of them where registers and LDS hold them.
    static constexpr int WPE = NP8 <= 9 && CT != CT_F8 && K != 7 ? 3 : 2;
    static constexpr int TH = !PRE ? 8 : (CT == CT_F8 || (WPE == 3 && CM != 1 && CT != CT_F32) ? 4 : 8) / (CM != 1 && (K == 7 || (CT == CT_F8 && NP8 == 16)) ? 2 : 1);
    static constexpr int UH = TH + K - 1;
    static constexpr int PITCH = !PRE ? 136 : (CT == CT_F8 ? 528 : (CT == CT_F32 ? 136 : 264));
    static constexpr int MAXLRX = !PRE ? 73 : (CT == CT_F8 ? 137 : (CT == CT_F32 ? 41 : 73)), MAXLRY = (UH - 1) / 2 + 5, NXC = (MAXLRX + 63) / 64;
    static constexpr int NLRP = (CM * MAXLRY + 3) / 4;
    static constexpr int NB16 = N16 * NMB, NB8 = N8 * NMB, NB32 = N2 * NMB;
    static_assert(CM * MAXLRY * MAXLRX <= CM * UH * PITCH, "the LR rows fit where the tile goes");
};

template <int CT> struct StoredAs;      // a coefficient in memory
template <> struct StoredAs<CT_F16> { typedef __half type; };
template <> struct StoredAs<CT_F32> { typedef float type; };
template <> struct StoredAs<CT_F8> { typedef f8e4m3 type; };
template <> struct StoredAs<CT_BF16> { typedef bf16raw type; };

constexpr float SLOT_LO = 2048.0f;       // scale of fp16's second part

template <int K, int CM, int CT, int NP8, int KIND, bool PRE>
__global__ __launch_bounds__(256, (SlotCfg<K, CM, CT, NP8, KIND, PRE>::WPE))
void k_assemble_slots(const SlotArgs a) {
    using F = SlotCfg<K, CM, CT, NP8, KIND, PRE>;
    constexpr bool LG = F::LG;
    constexpr int KK = F::KK, R = F::R, RH0 = F::RH0, NSLOT = F::NSLOT, NMB = F::NMB, P = F::P, NPART = F::NPART, NACC = F::NACC;
    constexpr int N16 = F::N16, N8 = F::N8, NLOAD = F::NLOAD, UH = F::UH, PITCH = F::PITCH, MAXLRX = F::MAXLRX, MAXLRY = F::MAXLRY, QG = F::QGP;
    constexpr unsigned CB = F::CB;

    __shared__ float U[CM * UH * PITCH];           // up-sampled tile; before that, in its place, the LR footprint
    __shared__ float V[CM * UH * MAXLRX];          // after the vertical pass
    __shared__ float4 wk[8];                          // Keys weights by phase numerator
    __shared__ float4 yw[UH];                         // a tile's rows: weights, first LR row
    __shared__ int yb[UH];
    __shared__ u32x4 A16[(N16 ? N16 : 1) * NMB * NPART * 64];
    __shared__ u32x2 A8[(N8 ? 1 : 0) * NMB * NPART * 64 + 1];
    __shared__ float A32[F::N2 * NMB * 64 + 1];
    __shared__ unsigned ptab[2 * NLOAD];              // byte offset of the plane each lane half loads
    __shared__ int ktab[8 * NP8];
    __shared__ float gtab[8 * NP8];
    __shared__ unsigned dmax[4];                      // bits of the dictionary's largest magnitude, of each wavefront's part
    float* const lrT = U;

    const int tid = threadIdx.x, lane = tid & 63, hf = lane >> 5, j = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = (int)blockIdx.x & ((1 << a.group_shift) - 1);
    const int t_end = min(a.ntiles, (grp + 1) * a.share);
    int t = grp * a.share + ((int)blockIdx.x >> a.group_shift);
    if (t >= t_end) return;
    // units of a tile row, column classes of the tile and the stride between them (planar: known when compiled)
    const int upr = PRE ? a.upr : 4 / P, sw = PRE ? a.sw : P, ng = PRE ? a.ng : 32 * (4 / P) + (K - 2) / P + 1;
    const int TW = 32 * P * upr;
    const int wb = PRE ? a.w : a.W;                   // pixels of a row of a coefficient plane
    const unsigned plane_b = (unsigned)a.H * (unsigned)a.W * CB;          // bytes of an atom's coefficients (below 4 GB for all of them)

    // (upr: units of a row of this tile; planar: those that hold any of the image)
    struct Tile { int n, Y0, X0, upr; };
    auto tile_of = [&](int i) -> Tile {
        const unsigned per = (unsigned)a.tiles_x * (unsigned)a.tiles_y, n = (unsigned)i / per, r = (unsigned)i - n * per;
        const unsigned ty = r / (unsigned)a.tiles_x;
        const int X0 = (int)(r - ty * (unsigned)a.tiles_x) * TW;
        return {(int)n, (int)ty * a.th, X0, PRE ? upr : min(upr, (wb - X0 + 32 * P - 1) / (32 * P))};
    };
    // ---- tables and operands, as in sr_mfma_kernel.h: everything is requested before anything is waited for
    auto load_atom = [&](int i, int h) -> int {
        return F::F32 ? 2 * i + h : (i < 8 * N16 ? 16 * (i >> 3) + 8 * h + (i & 7) : 16 * N16 + 4 * h + (i - 8 * N16));
    };
    if (!a.identity) {
        for (int e = tid; e < 8 * NP8; e += 256) {
            const int i = e < a.n_fold ? e : a.n_fold - 1;
            const int k = a.kept[i];
            const float g = a.gamma[i];
            ktab[e] = k;
            gtab[e] = g;
        }
        __syncthreads();
    }
    for (int e = tid; e < 2 * NLOAD; e += 256) {
        const int hh = e / NLOAD, at = load_atom(e - hh * NLOAD, hh);
        ptab[e] = (unsigned)(a.identity ? (at < a.n_fold ? at : a.n_fold - 1) : ktab[at]) * plane_b;
    }
    auto dict_entry = [&](int at, int tap) -> float {
        const int row = a.identity ? (at < a.n_fold ? at : a.n_fold - 1) : ktab[at];
        return a.dict[(unsigned)(row * KK + (tap < 0 ? 0 : tap))];
    };
    auto dict_value = [&](int at, int tap, float d) -> float {
        const float g = a.identity ? 1.0f : gtab[at];
        return tap < 0 || at >= a.n_fold ? 0.0f : g * d;
    };
    constexpr int M32 = (F::NB32 + 3) / 4, M16 = (F::NB16 + 3) / 4, M8 = (F::NB8 + 3) / 4;
    float dv32[M32 ? M32 : 1], dv16[M16 ? M16 : 1][8], dv8[M8 ? M8 : 1][4];
#pragma unroll
    for (int m = 0; m < M32; ++m) {
        const int blk = wave + 4 * m < F::NB32 ? wave + 4 * m : F::NB32 - 1, mb = blk % NMB, st = blk / NMB;
        dv32[m] = dict_entry(2 * st + hf, tap_of_row<K>(j, mb));
    }
#pragma unroll
    for (int m = 0; m < M16; ++m) {
        const int blk = wave + 4 * m < F::NB16 ? wave + 4 * m : F::NB16 - 1, mb = blk % NMB, c16 = blk / NMB;
#pragma unroll
        for (int i = 0; i < 8; ++i) dv16[m][i] = dict_entry(16 * c16 + 8 * hf + i, tap_of_row<K>(j, mb));
    }
#pragma unroll
    for (int m = 0; m < M8; ++m) {
        const int mb = wave + 4 * m < F::NB8 ? wave + 4 * m : F::NB8 - 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) dv8[m][i] = dict_entry(16 * N16 + 4 * hf + i, tap_of_row<K>(j, mb));
    }

    // LR footprint of a tile -> registers (raw bits): wavefront w takes the (channel, row) pairs w, w + 4, ...; the lane is the column
    unsigned lrv[F::NLRP][F::NXC];
    auto load_lr = [&](const Tile tp) {
        const TileOrigin o = tile_origin(tp.Y0, tp.X0, R, a.th + K - 1, TW + K - 1, a.H, a.W, a.s);
        const char* img = (const char*)a.lr + (size_t)tp.n * a.C * ((size_t)a.h * a.w * (a.io_f16 ? 2 : 4));
        unsigned xo[F::NXC];
#pragma unroll
        for (int xc = 0; xc < F::NXC; ++xc) xo[xc] = (unsigned)clampi(o.lx0 + lane + 64 * xc, 0, a.w - 1);
#pragma unroll
        for (int u = 0; u < F::NLRP; ++u) {
            const int p = wave + 4 * u, c = p / MAXLRY, ry = p - c * MAXLRY;
            const unsigned row = ((unsigned)(c < a.C ? c : 0) * (unsigned)a.h + (unsigned)clampi(o.ly0 + ry, 0, a.h - 1)) * (unsigned)a.w;
#pragma unroll
            for (int xc = 0; xc < F::NXC; ++xc) {
                if (a.io_f16) lrv[u][xc] = *(const unsigned short*)(img + (size_t)(row + xo[xc]) * 2);
                else lrv[u][xc] = *(const unsigned*)(img + (size_t)(row + xo[xc]) * 4);
            }
        }
    };

    // A unit of a tile: its row, the first pixel of its words in a coefficient row, its sub-pixel column (planar: none)
    struct Unit { int row, x, jx, col; };             // (col: its first group of columns in the tile)
    auto unit_of = [&](const Tile tp, int u) -> Unit {
        int row = 0, r = u;
        while (r >= tp.upr) { r -= tp.upr; ++row; }                        // (at most 32 units)
        return PRE ? Unit{row, tp.X0 / a.s, r, 0} : Unit{row, tp.X0 + 32 * P * r, 0, 32 * r};
    };
    unsigned raw[NLOAD], pix = 0u, sh = 0u;
    const char* cimg = nullptr;
    // where the lane's words of a unit lie; a word that would stick out of its row is taken from the row's end and shifted
    auto point_at = [&](const Tile tp, const Unit un) {
        const int y = min(tp.Y0 + un.row, a.H - 1), x = un.x + P * j, xc = x + P <= wb ? x : wb - P;
        sh = x < wb ? (unsigned)(x - xc) * 8u * CB : 0u;
        unsigned at;
        if constexpr (PRE) {
            int ly, iy;
            divmod_scale(y, a.s, ly, iy);
            at = (unsigned)(iy * a.s + un.jx) * ((unsigned)a.h * (unsigned)a.w) + (unsigned)ly * (unsigned)a.w + (unsigned)xc;
        } else {
            at = (unsigned)y * (unsigned)a.W + (unsigned)xc;
        }
        pix = at * CB;
        cimg = (const char*)a.coeff + (size_t)tp.n * a.L * ((size_t)a.H * a.W * CB);
    };
    struct __attribute__((packed, aligned(1))) Word { unsigned v; };       // (of the coefficients' own alignment)
    const unsigned* const pt = ptab + hf * NLOAD;
    auto load_word = [&](int i) -> unsigned { return ((const Word*)(cimg + (size_t)(pix + pt[i])))->v; };

    Tile cur = tile_of(t);
    load_lr(cur);
    __syncthreads();                                                       // the table of plane offsets is written
    if (wave < a.th * cur.upr) {
        point_at(cur, unit_of(cur, wave));
#pragma unroll
        for (int i = 0; i < NLOAD; ++i) raw[i] = load_word(i);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (tid < 2 * a.s) {
        float wt[4];
        keys_weights(tid, a.s, wt);
        wk[tid] = make_float4(wt[0], wt[1], wt[2], wt[3]);
    }
#pragma unroll
    for (int m = 0; m < M32; ++m) {
        const int blk = wave + 4 * m, mb = blk % NMB, st = blk / NMB;
        if (blk < F::NB32) A32[blk * 64 + lane] = dict_value(2 * st + hf, tap_of_row<K>(j, mb), dv32[m]);
    }
    // the values of the operands, and (SCALED) the exponent of the power of two that the dictionary is multiplied by
#pragma unroll
    for (int m = 0; m < M16; ++m) {
        const int blk = wave + 4 * m < F::NB16 ? wave + 4 * m : F::NB16 - 1, mb = blk % NMB, c16 = blk / NMB;
#pragma unroll
        for (int i = 0; i < 8; ++i) dv16[m][i] = dict_value(16 * c16 + 8 * hf + i, tap_of_row<K>(j, mb), dv16[m][i]);
    }
#pragma unroll
    for (int m = 0; m < M8; ++m) {
        const int mb = wave + 4 * m < F::NB8 ? wave + 4 * m : F::NB8 - 1;
#pragma unroll
        for (int i = 0; i < 4; ++i) dv8[m][i] = dict_value(16 * N16 + 4 * hf + i, tap_of_row<K>(j, mb), dv8[m][i]);
    }
    int scale = 0;
    if constexpr (F::SCALED) {
        unsigned m = 0u;
#pragma unroll
        for (int b = 0; b < M16; ++b)
#pragma unroll
            for (int i = 0; i < 8; ++i) m = max(m, __float_as_uint(fabsf(dv16[b][i])));
#pragma unroll
        for (int b = 0; b < M8; ++b)
#pragma unroll
            for (int i = 0; i < 4; ++i) m = max(m, __float_as_uint(fabsf(dv8[b][i])));
        m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xf, 0xf, false));       // neighbours, pairs, quads, halves of a row
        m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xf, 0xf, false));
        m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xf, 0xf, false));
        m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x140, 0xf, 0xf, false));
        m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x142, 0xa, 0xf, false));      // rows 1 and 3 from the row before, then
        m = max(m, (unsigned)__builtin_amdgcn_update_dpp(0, (int)m, 0x143, 0xc, 0xf, false));      // the upper half from lane 31: lane 63 has all
        if (lane == 63) dmax[wave] = m;
        __syncthreads();
        const unsigned all = max(max(dmax[0], dmax[1]), max(dmax[2], dmax[3]));
        scale = 14 + 127 - (int)(__builtin_amdgcn_readfirstlane(all) >> 23);
    }
    auto scaled = [&](float v) -> float { return F::SCALED ? ldexpf(v, scale) : v; };
    // N dictionary values as NPART operands
    auto parts = [&](auto& dst, int blk, const auto& d) {
        using Vec = typename std::remove_reference<decltype(dst[0])>::type;
        constexpr int N = sizeof(Vec) / 2;
        unsigned short b[NPART][N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if constexpr (F::BF) {
                float rest = d[i];
#pragma unroll
                for (int p = 0; p < NPART; ++p) {
                    const __bf16 v = (__bf16)rest;
                    rest -= (float)v;
                    b[p][i] = __builtin_bit_cast(unsigned short, v);
                }
            } else if constexpr (!F::F32) {
                const _Float16 v = (_Float16)d[i];
                b[0][i] = __builtin_bit_cast(unsigned short, v);
                b[1][i] = __builtin_bit_cast(unsigned short, (_Float16)((d[i] - (float)v) * (NACC == 2 ? SLOT_LO : 1.0f)));
            }
        }
#pragma unroll
        for (int p = 0; p < NPART; ++p) {
            Vec v;
#pragma unroll
            for (int i = 0; i < N / 2; ++i) v[i] = (unsigned)b[p][2 * i] | ((unsigned)b[p][2 * i + 1] << 16);
            dst[(blk * NPART + p) * 64 + lane] = v;
        }
    };
    if constexpr (!F::F32) {
#pragma unroll
        for (int m = 0; m < M16; ++m) {
            const int blk = wave + 4 * m, mb = blk % NMB, c16 = blk / NMB;
            if (blk < F::NB16) {
                const bool ones = LG && sum_row<K>(j, mb);                 // logits: this row sums the exponentials
                float d[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int at = 16 * c16 + 8 * hf + i;
                    d[i] = ones ? (at < a.n_fold ? 1.0f : 0.0f) : scaled(dv16[m][i]);
                }
                parts(A16, blk, d);
            }
        }
#pragma unroll
        for (int m = 0; m < M8; ++m) {
            const int mb = wave + 4 * m;
            if (mb < F::NB8) {
                const bool ones = LG && sum_row<K>(j, mb);
                float d[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int at = 16 * N16 + 4 * hf + i;
                    d[i] = ones ? (at < a.n_fold ? 1.0f : 0.0f) : scaled(dv8[m][i]);
                }
                parts(A8, mb, d);
            }
        }
    }

    const unsigned plane_px = (unsigned)a.H * (unsigned)a.W;
    for (;;) {
        // ---- stage 1: LR rows -> LDS, vertical pass, horizontal pass into the tile
        const TileOrigin o = tile_origin(cur.Y0, cur.X0, R, a.th + K - 1, TW + K - 1, a.H, a.W, a.s);
#pragma unroll
        for (int u = 0; u < F::NLRP; ++u) {
            const int p = wave + 4 * u;
            if (p < CM * MAXLRY) {
#pragma unroll
                for (int xc = 0; xc < F::NXC; ++xc)
                    if (lane + 64 * xc < MAXLRX)
                        lrT[p * MAXLRX + lane + 64 * xc] = a.io_f16 ? __half2float(__ushort_as_half((unsigned short)lrv[u][xc])) : __uint_as_float(lrv[u][xc]);
            }
        }
        const int rows = a.th + K - 1;
        if (tid < rows) {
            int m;
            const int f = src_floor(clampi(cur.Y0 - R + tid, 0, a.H - 1), a.s, m);
            float wt[4];
            keys_weights(m, a.s, wt);
            yw[tid] = make_float4(wt[0], wt[1], wt[2], wt[3]);
            yb[tid] = clampi(f - 1 - o.ly0, 0, MAXLRY - 4) * MAXLRX;
        }
        __syncthreads();
        // (row of a channel, footprint column) dealt to the threads with no idle lanes, four at a time so that their reads overlap
        static_assert(CM * UH * MAXLRX * MAXLRX <= (1 << 22) && CM * UH <= 1024, "item index beyond the exact range of the division");
        const int nlx = o.nlx < 4 ? 4 : o.nlx, items = a.C * rows * nlx;
        const unsigned inv = ((1u << 22) + nlx - 1) / nlx;
        for (int base = tid; base < items; base += 4 * 256) {
            float v[4][4];
            float4 w4[4];
            int dst[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int idx = base + 256 * k, idc = idx < items ? idx : items - 1;
                const int pr = (int)(((unsigned)idc * inv) >> 22), rx = idc - pr * nlx;
                const int c = pr >= 2 * rows ? 2 : (pr >= rows ? 1 : 0), yy = pr - c * rows;
                w4[k] = yw[yy];
                const float* const src = lrT + c * (MAXLRY * MAXLRX) + yb[yy] + rx;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[k][i] = src[i * MAXLRX];
                dst[k] = idx < items ? (c * UH + yy) * MAXLRX + rx : -1;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float wt[4] = {w4[k].x, w4[k].y, w4[k].z, w4[k].w};
                if (dst[k] >= 0) V[dst[k]] = dot4(wt, v[k][0], v[k][1], v[k][2], v[k][3]);
            }
        }
        __syncthreads();
        // a thread: a column of a channel, its weights in registers
        const int UW = TW + K - 1;
        for (int i = tid; i < a.C * UW; i += 256) {
            const int c = i >= 2 * UW ? 2 : (i >= UW ? 1 : 0), xx = i - c * UW;
            int m;
            const int f = src_floor(clampi(cur.X0 - R + xx, 0, a.W - 1), a.s, m);
            const float4 w4 = wk[m];
            const float wt[4] = {w4.x, w4.y, w4.z, w4.w};
            const unsigned g = PRE ? ((unsigned)xx * a.inv_sw) >> 16 : (unsigned)xx / P;
            const float* const src = V + c * (UH * MAXLRX) + clampi(f - 1 - o.lx0, 0, MAXLRX - 4);
            float* const dst = U + c * (UH * PITCH) + ((unsigned)xx - g * sw) * ng + g;
            constexpr int RB = 6;                                          // rows whose reads overlap
#pragma unroll
            for (int y0 = 0; y0 < UH; y0 += RB)
                if (y0 < rows) {
                    float v[RB][4];
#pragma unroll
                    for (int r = 0; r < RB; ++r)
                        if (y0 + r < UH) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) v[r][k] = src[(y0 + r) * MAXLRX + k];
                        }
#pragma unroll
                    for (int r = 0; r < RB; ++r)
                        if (y0 + r < UH) dst[(y0 + r) * PITCH] = dot4(wt, v[r][0], v[r][1], v[r][2], v[r][3]);
                }
        }
        __syncthreads();
        const bool more = t + a.stride < t_end;
        const Tile nxt = more ? tile_of(t + a.stride) : cur;
        if (more) load_lr(nxt);

        const int units = a.th * cur.upr;
        // A wavefront's first words of the next tile are requested with its last unit of this one.  The last tile of a row can have fewer
        // units than wavefronts: one that has none here requests them now.
        if constexpr (!PRE && P < 4) {
            if (more && wave >= units) {
                point_at(nxt, unit_of(nxt, wave));
#pragma unroll
                for (int i = 0; i < NLOAD; ++i) raw[i] = load_word(i);
            }
        }
        for (int u = wave; u < units; u += 4) {
            const Unit un = unit_of(cur, u);
            const unsigned ush = sh;
            // the next unit's words go into the registers that fall free: this tile's, or the next tile's first
            const bool tile_done = u + 4 >= units, fetch = more || !tile_done;
            if (tile_done) point_at(nxt, unit_of(nxt, wave));
            else point_at(cur, unit_of(cur, u + 4));
            if (__builtin_amdgcn_ballot_w64(ush != 0u)) {
#pragma unroll
                for (int i = 0; i < NLOAD; ++i) raw[i] >>= ush;
            }
            // logits: -max * log2(e) of the lane's pixels, over all planes (both lane halves)
            float nm[P];
            if constexpr (LG) {
                typedef _Float16 h2 __attribute__((ext_vector_type(2)));
                if constexpr (CT == CT_F32) {
                    float mx = __uint_as_float(raw[0]);
#pragma unroll
                    for (int i = 1; i < NLOAD; ++i) mx = fmaxf(mx, __uint_as_float(raw[i]));
                    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
                    nm[0] = logit_shift(fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])));
                } else {
                    h2 mx = __builtin_bit_cast(h2, raw[0]);
#pragma unroll
                    for (int i = 1; i < NLOAD; ++i) mx = pk_max_f16(mx, __builtin_bit_cast(h2, raw[i]));
                    const unsigned bits = __builtin_bit_cast(unsigned, mx);
                    const auto sw = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
                    mx = pk_max_f16(__builtin_bit_cast(h2, (unsigned)sw[0]), __builtin_bit_cast(h2, (unsigned)sw[1]));
                    const unsigned both = __builtin_bit_cast(unsigned, mx);
                    if constexpr (P == 2) {
#pragma unroll
                        for (int q = 0; q < 2; ++q)
                            nm[q] = CT == CT_BF16 ? logit_shift(__uint_as_float((both >> (16 * q)) << 16)) : logit_shift((float)mx[q]);
                    }
                }
            }
            // a pair of atoms of slot q as an operand word
            auto pair = [&](unsigned even, unsigned odd, int q) -> unsigned {
                if constexpr (LG && CT == CT_F32) {
                    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
                    typedef float f2 __attribute__((ext_vector_type(2)));
                    const f2 e = {logit_exp(__uint_as_float(even), nm[0]), logit_exp(__uint_as_float(odd), nm[0])};
                    return __builtin_bit_cast(unsigned, __builtin_convertvector(e, h2));
                } else if constexpr (LG) {
                    return exp_pair<CT == CT_BF16>(even, odd, q, nm[q]);
                } else if constexpr (CT == CT_F8) {
                    const unsigned both = __builtin_amdgcn_perm(odd, even, q < 2 ? 0x05010400u : 0x07030602u);
                    return widen_pair(both, q);
                } else {
                    return pack_pair(even, odd, q);
                }
            };
            const int y = cur.Y0 + un.row;
            const int x0 = un.x + P * j;                                   // of the lane's first slot, in a coefficient row
            const unsigned out_px = (unsigned)a.C * plane_px;
            const __amdgpu_buffer_rsrc_t out_rsrc = __builtin_amdgcn_make_buffer_rsrc(
                (char*)a.out + (size_t)cur.n * ((size_t)out_px * (a.io_f16 ? 2 : 4)), 0, (int)(out_px * (a.io_f16 ? 2u : 4u)), RAW_BUFFER);
            constexpr unsigned BEYOND = 0xffffffc0u;                       // (no image ends there, see slots_supported)
            const int se = PRE ? a.s : 1;
            // Half 1 has one filter row less: its last one meets weights that are zero, and reads a row of the patch again (a row further
            // down may hold what no weight of zero makes harmless).
            const float* const ub = U + (un.row + hf * RH0) * PITCH + j + un.col;
            const float* const ub_last = ub + (RH0 - 1 - hf) * PITCH;
#pragma unroll
            for (int q0 = 0; q0 < P; q0 += QG) {
                const bool last_pass = q0 + QG >= P;
                f32x16 acc[QG][NMB][NACC];
#pragma unroll
                for (int q = 0; q < QG; ++q)
#pragma unroll
                    for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                        for (int n = 0; n < NACC; ++n)
#pragma unroll
                            for (int v = 0; v < 16; ++v) acc[q][mb][n][v] = 0.0f;
                if constexpr (F::F32) {
#pragma unroll
                    for (int st = 0; st < F::N2; ++st) {               // (a multiple of four)
#pragma unroll
                        for (int mb = 0; mb < NMB; ++mb)
                            acc[0][mb][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(A32[(st * NMB + mb) * 64 + lane], __uint_as_float(raw[st]), acc[0][mb][0], 0, 0, 0);
                        if ((st & 3) == 3) {
                            __builtin_amdgcn_sched_barrier(0);
                            if (fetch) {
#pragma unroll
                                for (int i = st - 3; i <= st; ++i) raw[i] = load_word(i);
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                } else {
#pragma unroll
                    for (int c16 = 0; c16 < N16; ++c16) {
#pragma unroll
                        for (int q = 0; q < QG; ++q) {
                            u32x4 bw;
#pragma unroll
                            for (int m = 0; m < 4; ++m) bw[m] = pair(raw[8 * c16 + 2 * m], raw[8 * c16 + 2 * m + 1], q0 + q);
#pragma unroll
                            for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                                for (int p = 0; p < NPART; ++p)
                                    acc[q][mb][p < NACC ? p : 0] = mfma_16<F::BF>(A16[((c16 * NMB + mb) * NPART + p) * 64 + lane], bw, acc[q][mb][p < NACC ? p : 0]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        if (last_pass && fetch) {
#pragma unroll
                            for (int i = 0; i < 8; ++i) raw[8 * c16 + i] = load_word(8 * c16 + i);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if constexpr (N8 != 0) {
#pragma unroll
                        for (int q = 0; q < QG; ++q) {
                            u32x2 bw;
#pragma unroll
                            for (int m = 0; m < 2; ++m) bw[m] = pair(raw[8 * N16 + 2 * m], raw[8 * N16 + 2 * m + 1], q0 + q);
#pragma unroll
                            for (int mb = 0; mb < NMB; ++mb)
#pragma unroll
                                for (int p = 0; p < NPART; ++p)
                                    acc[q][mb][p < NACC ? p : 0] = mfma_8<F::BF>(A8[(mb * NPART + p) * 64 + lane], bw, acc[q][mb][p < NACC ? p : 0]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                        if (last_pass && fetch) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) raw[8 * N16 + i] = load_word(8 * N16 + i);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                // stage 4: each half filters its taps, channel by channel; the halves' sums are exchanged and stored
                float rsum[QG];
#pragma unroll
                for (int q = 0; q < QG; ++q) {
                    if constexpr (NACC == 2) {
#pragma unroll
                        for (int v = 0; v < NSLOT + (LG ? 1 : 0); ++v)
                            acc[q][v / 16][0][v % 16] = fmaf(acc[q][v / 16][1][v % 16], 1.0f / SLOT_LO, acc[q][v / 16][0][v % 16]);
                    }
                    rsum[q] = 1.0f;
                    if constexpr (LG) rsum[q] = 1.0f / acc[q][NSLOT / 16][0][NSLOT % 16];
                }
                unsigned at[QG][K];
#pragma unroll
                for (int q = 0; q < QG; ++q)
#pragma unroll
                    for (int dx = 0; dx < K; ++dx) {
                        const unsigned e = (unsigned)(se * (q0 + q) + (PRE ? un.jx : 0) + dx);                   // scalar
                        const unsigned g = PRE ? (e * a.inv_sw) >> 16 : e / P;
                        at[q][dx] = (e - g * (unsigned)sw) * (unsigned)ng + g;
                    }
                // Every lane stores, for every channel that there is room for: what is outside the image goes where the buffer drops it.
                // Behind a branch the compiler cannot count the stores, and the next unit, which waits for loads issued before them,
                // waits for them as well.
                constexpr int NS = QG == 4 ? 2 : 1;                        // pixels a lane stores: half hf has slots NS hf + i (one slot: half 0)
                unsigned odd = 0u;                                         // bit c NS + i: what the lane stores there is not finite
#pragma unroll
                for (int c = 0; c < CM; ++c) {
                        float sum[QG];
#pragma unroll
                        for (int q = 0; q < QG; ++q) {
                            // (row by row, as the streaming kernel: the same sums where the fold is the same)
                            sum[q] = 0.0f;
#pragma unroll
                            for (int v = 0; v < NSLOT; ++v) {
                                const int dy = v / K, dx = v % K;
                                const float u = dy + 1 < RH0 ? ub[at[q][dx] + (c * UH + dy) * PITCH] : ub_last[at[q][dx] + c * UH * PITCH];
                                sum[q] = fmaf(acc[q][v / 16][0][v % 16], u, sum[q]);
                            }
                            if constexpr (LG) sum[q] *= rsum[q];
                            if constexpr (F::SCALED) sum[q] = ldexpf(sum[q], -scale);
                        }
#pragma unroll
                        for (int i = 0; i < NS; ++i) {
                            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum[i]), __float_as_uint(sum[QG == 1 ? 0 : i + NS]), false, false);
                            const float v = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
                            const int x = x0 + q0 + (QG == 1 ? 0 : NS * hf + i);
                            const bool valid = y < a.H && x < wb && (QG != 1 || hf == 0) && c < a.C;
                            const unsigned px = (unsigned)c * plane_px + (unsigned)y * (unsigned)a.W + (unsigned)(se * x + un.jx);
                            if (a.io_f16) store16(out_rsrc, valid ? 2u * px : BEYOND, v);
                            else store32(out_rsrc, valid ? 4u * px : BEYOND, __float_as_uint(v));
                            if constexpr (!F::ST) odd |= valid && __builtin_amdgcn_classf(v, 0x207) ? 1u << (c * NS + i) : 0u;      // NaN, infinity
                        }
                    }
                // An infinite coefficient, logit, image value or dictionary entry meets the zeros of the padding and the dictionary's second part here and gives
                // NaN also where the plain sums give infinity, or a number (logits).  Such pixels are taken again, one by one, as in the generic kernel.
                if constexpr (!F::ST)
                    if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd != 0u) != 0, 0)) {
                        using TC = typename StoredAs<CT>::type;
#pragma unroll 1
                        for (int i = 0; i < NS; ++i) {
                            const int q = q0 + (QG == 1 ? 0 : NS * hf + i), x = x0 + q;
                            const bool mine = ((odd >> i) & (NS == 2 ? 0x15u : 0x7u)) != 0u;
                            unsigned at = 0u;                              // the pixel's place in a coefficient plane
                            if (mine) {
                                if constexpr (PRE) {
                                    int ly, iy;
                                    divmod_scale(y, a.s, ly, iy);
                                    at = (unsigned)(iy * a.s + un.jx) * ((unsigned)a.h * (unsigned)a.w) + (unsigned)ly * (unsigned)a.w + (unsigned)x;
                                } else {
                                    at = (unsigned)y * (unsigned)a.W + (unsigned)x;
                                }
                            }
                            const TC* const base = (const TC*)a.coeff + (size_t)cur.n * a.L * plane_px + at;
                            auto stored = [&](int atom) -> float { return ld_as_float(base, (size_t)atom * plane_px); };
                            float Fk[KK], esum = 0.0f, shift = 0.0f;
#pragma unroll
                            for (int t = 0; t < KK; ++t) Fk[t] = 0.0f;
                            if constexpr (LG) {
                                float m = stored(0);
#pragma unroll 4
                                for (int l = 1; l < a.n_fold; ++l) m = fmaxf(m, stored(l));
                                shift = logit_shift(m);
                            }
                            constexpr int NB = 8;                          // coefficients requested together
#pragma unroll 1
                            for (int l0 = 0; l0 < a.n_fold; l0 += NB) {
                                float phi[NB];
#pragma unroll
                                for (int b = 0; b < NB; ++b) {
                                    const int l = l0 + b < a.n_fold ? l0 + b : a.n_fold - 1;
                                    phi[b] = stored(a.kept[l]) * a.gamma[l];
                                }
#pragma unroll
                                for (int b = 0; b < NB; ++b)
                                    if (l0 + b < a.n_fold) {               // wave-uniform
                                        float p = phi[b];
                                        if constexpr (LG) {
                                            p = __half2float(__float2half_rn(logit_exp(p, shift)));
                                            esum += p;
                                        }
                                        const float* const d = a.dict + (size_t)a.kept[l0 + b] * KK;
#pragma unroll
                                        for (int t = 0; t < KK; ++t) Fk[t] = fmaf(p, d[t], Fk[t]);
                                    }
                            }
#pragma unroll 1
                            for (int c = 0; c < a.C; ++c) {
                                float v = 0.0f;
#pragma unroll
                                for (int dy = 0; dy < K; ++dy)
#pragma unroll
                                    for (int dx = 0; dx < K; ++dx) {
                                        const unsigned e = (unsigned)(se * q + (PRE ? un.jx : 0) + dx), g = PRE ? (e * a.inv_sw) >> 16 : e / P;
                                        v = fmaf(Fk[dy * K + dx], U[(c * UH + un.row + dy) * PITCH + j + un.col + (e - g * (unsigned)sw) * (unsigned)ng + g], v);
                                    }
                                if constexpr (LG) v = v * (1.0f / esum);
                                const bool again = ((odd >> (c * NS + i)) & 1u) != 0u;
                                const unsigned px = (unsigned)c * plane_px + (unsigned)y * (unsigned)a.W + (unsigned)(se * x + un.jx);
                                if (a.io_f16) store16(out_rsrc, again ? 2u * px : BEYOND, v);
                                else store32(out_rsrc, again ? 4u * px : BEYOND, __float_as_uint(v));
                            }
                        }
                    }
            }
        }
        if (!more) break;
        t += a.stride;
        cur = nxt;
        __syncthreads();                                                   // every wavefront is done with this tile
    }
}

template <int K, int CM, int CT, int NP8, int KIND, bool PRE>
static hipError_t launch_slots_p(const AssembleArgs& c, const LaunchTo& st) {
    using F = SlotCfg<K, CM, CT, NP8, KIND, PRE>;
    SlotArgs a;
    a.lr = c.lr; a.coeff = c.coeff; a.dict = c.dict; a.out = c.out;
    a.N = c.N; a.C = c.C; a.h = c.h; a.w = c.w; a.H = c.H; a.W = c.W; a.s = c.s; a.L = c.L;
    a.n_fold = c.n_fold; a.io_f16 = c.io_f16; a.identity = c.identity;
    a.upr = PRE ? a.s : 4 / F::P;                      // planar: tiles of 128 columns
    a.sw = F::P * (PRE ? a.s : 1);
    a.ng = 32 * a.upr * F::P / a.sw + (K - 2) / a.sw + 1;
    a.inv_sw = (65536u + (unsigned)a.sw - 1) / (unsigned)a.sw;
    const int tw = 32 * F::P * a.upr, cus = units_of(c), cap = F::WPE * cus;
    a.tiles_x = (a.W + tw - 1) / tw;
    // Rows of a tile, by the cycles of the fullest CU's SIMDs: units of a wavefront (matrix instructions and filtering) and the
    // up-sampling of th + K - 1 rows, times its tiles; or, where that is more, what a workgroup's tiles take one after the other with the
    // latencies that nothing hides.  (One to eight rows, one run, us: fp32 7x7 716 x 404 x1 103 atoms 34 / 50 with two / eight, 1080
    // x 1020 x3 fp16 72 atoms 71 / 51 with eight / four.)
    constexpr long long mfma = F::F32 ? 64ll * F::N2 * F::NMB : 32ll * F::P * F::NMB * F::NPART * (F::N16 + F::N8);
    const long long unit = mfma + F::P * (8ll * a.C * F::NSLOT + 250);
    long long best = 0;
    for (int th = 1; th <= F::TH; th *= 2) {
        const long long tiles = (long long)a.tiles_x * ((a.H + th - 1) / th) * a.N, rounds = (tiles + cap - 1) / cap;
        const long long of_a_cu = rounds == 1 ? (tiles + cus - 1) / cus : rounds * F::WPE;
        const long long units = (th * a.upr + 3) / 4, stage1 = 60ll * (th + K - 1) * tw * a.C / 256;
        const long long busy = of_a_cu * (units * unit + stage1), alone = rounds * (units * (unit + 2000) + stage1 + 5000);
        const long long cost = busy > alone ? busy : alone;
        if (th == 1 || cost <= best) { best = cost; a.th = th; }
    }
    a.tiles_y = (a.H + a.th - 1) / a.th;
    const long long nt = (long long)a.tiles_x * a.tiles_y * a.N;
    if (nt > 0x3fffffffLL) return hipErrorInvalidValue;
    a.ntiles = (int)nt;
    const int blocks = nt < cap ? (int)nt : cap;
    a.group_shift = blocks % 8 == 0 ? 3 : 0;
    const int groups = 1 << a.group_shift;
    a.share = (a.ntiles + groups - 1) / groups;
    a.stride = blocks / groups;
    if (st.walk) {
        *st.walk = {1, tw, a.th, a.ntiles, blocks, 4};
        return hipSuccess;
    }
    memcpy(a.kept, c.kept, sizeof(a.kept));
    memcpy(a.gamma, c.gamma, sizeof(a.gamma));
    hipLaunchKernelGGL((k_assemble_slots<K, CM, CT, NP8, KIND, PRE>), dim3(blocks), dim3(256), 0, st.stream, a);
    return hipGetLastError();
}

template <int K, int CM, int CT, int NP8, int KIND>
static hipError_t launch_slots_n(const AssembleArgs& a, const LaunchTo& st) {
    if constexpr (KIND != SLOT_STREAMED)
        return a.pre_shuffle ? launch_slots_p<K, CM, CT, NP8, KIND, true>(a, st) : launch_slots_p<K, CM, CT, NP8, KIND, false>(a, st);
    else if constexpr (NP8 == 16 || (CT == CT_F8 ? K == 7 : CT == CT_F32 || K != 5 || CM == 1))      // (what slots_faster sends here)
        return a.pre_shuffle ? hipErrorInvalidValue : launch_slots_p<K, CM, CT, NP8, KIND, false>(a, st);
    else if constexpr (K == 5 && CM == 3 && (CT == CT_F16 || CT == CT_BF16))
        return a.pre_shuffle ? launch_slots_p<K, CM, CT, NP8, KIND, true>(a, st) : launch_slots_p<K, CM, CT, NP8, KIND, false>(a, st);
    else
        return hipErrorInvalidValue;
}

template <int K, int CM, int CT, int KIND>
static hipError_t launch_slots_k(const AssembleArgs& a, const LaunchTo& st) {
    if (a.n_fold <= 32) return launch_slots_n<K, CM, CT, 4, KIND>(a, st);
    if (a.n_fold <= 72) return launch_slots_n<K, CM, CT, 9, KIND>(a, st);
    return launch_slots_n<K, CM, CT, 16, KIND>(a, st);
}

template <int K, int CM, int CT>
static hipError_t launch_slots_v(const AssembleArgs& a, bool streamed, const LaunchTo& st) {
    if (streamed) return launch_slots_k<K, CM, CT, SLOT_STREAMED>(a, st);
    if constexpr (CT != CT_F8)
        if (a.logits) return launch_slots_k<K, CM, CT, SLOT_LOGITS>(a, st);
    return launch_slots_k<K, CM, CT, SLOT_VALUES>(a, st);
}

template <int K, int CM>
static hipError_t launch_slots_t(const AssembleArgs& a, bool streamed, const LaunchTo& st) {
    switch (a.coeff_dtype) {
    case SR_F16:  return launch_slots_v<K, CM, CT_F16>(a, streamed, st);
    case SR_BF16: return launch_slots_v<K, CM, CT_BF16>(a, streamed, st);
    case SR_F32:  return launch_slots_v<K, CM, CT_F32>(a, streamed, st);
    default:      return launch_slots_v<K, CM, CT_F8>(a, streamed, st);
    }
}
}  // namespace srd
