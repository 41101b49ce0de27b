// Forward and backward-data convolution of layers of any channel count,
// filter, image size and stride on gfx950 matrix cores: a blocked implicit
// GEMM with both operands staged in LDS (Eqs. (1) and (3) of Sec. II-A on the
// tile of Sec. III-A).
//
//   D[o][pixel] = sum over (tap, input channel) of A[o][tap, ci] * B[tap, ci][pixel]
//
// Work split.  A workgroup of four waves computes OB output channels of a
// block of BU x BV output pixels of one image, flattened: pixel p of the block
// is MFMA column p, so narrow images (7 to 56 columns) fill the columns that a
// fixed 64-wide strip leaves empty.  The input channels are walked in chunks
// of 8 CCG; the next chunk's global loads are issued before the MFMA loop of
// the present one and written to LDS after it, and two workgroups share a
// CU, so that one computes while the other stages.
//
// LDS layout.  Both operands lie as 16-byte records of eight channels (what a
// lane of v_mfma_f32_32x32x16_bf16 reads): weights [plane][tap][group][o],
// the input patch [row][column][plane, group] with an odd number of records a
// pixel (conflict-free reads of neighbouring pixels).  The tap's shift is an
// offset common to all lanes.  At input stride 2 even and odd columns lie
// apart, so that the pixels of a tap are neighbours again.  NCHW rows are
// transposed on the way in: 16-byte loads of 8 channels, one byte permute per
// two values.
//
// fp32 layers run on the same matrix instruction.  A value from 2^-110 on is
// split into three bf16 parts that add up to it exactly (three roundings to
// nearest, 24 bits), and the product is formed from six part products (parts
// 0*0, 0*1, 1*0, 1*1, 0*2, 2*0); the three left out come to at most 2^-24 of a
// product, 2^-26 as a rule, of random sign.  Where it took over in 160 fp32 layers
// of mesh models, the error against 64 bits is 0.64 (forward) and 0.69 (input
// gradient) of the fp32 instruction's (geometric means; no layer above it): 16
// channels are added in eight steps there, in six here.  With the products of
// parts 1*2 and 2*1 as well no layer's error changed by 1 %, at 2 to 5 % more
// time.  Six bf16 MFMAs take 16 channels in 192 cycles; v_mfma_f32_32x32x2_f32
// takes 512.  A block that meets values the parts cannot hold (infinities, NaN,
// magnitudes near the ends of the range) is computed once more on the fp32
// instruction, from the same staging, for the outputs that read them.
//
// Bound: the matrix cores at many channels; what holds it is staging (waits
// for loads and barriers, 2 waves per SIMD).  Measured against the chunked
// kernel it replaces for these layers (us a pass): 128 -> 128 channels 3x3 on
// 32 images of 28x28, bf16: 131 -> 21; 256 -> 256 3x3 stride 2 on 28x28:
// forward 286 -> 35, backward-data 274 -> 33; fp32 128 -> 128 3x3 on a 64x64
// tile: 208 -> 28 and 210 -> 24; fp32 32 -> 32 stride 2 on a 512x512 tile,
// backward-data: 89 -> 17.
#pragma once

#include <hip/hip_runtime.h>

#include "bf16util.h"
#include "kernels.h"

namespace dc {

static constexpr int kTileThreads = 256;
static constexpr int kTileWord3 = 0x00020000;   // buffer resource word 3 (gfx9 family: raw access)
// Byte offset past every buffer here, whatever channel offset is added (the
// plan keeps those below 2^31): such a load returns 0, such a store is dropped.
static constexpr uint32_t kTileOut = 0x80000000u;
static constexpr int kTileNT = 2;               // a buffer store's non-temporal bit
static constexpr int kTileRedoBytes = 16;       // fp32: LDS of the redo word, past the records

// weight staging: per-element gathers (any layout); forward, a thread's 8
// channels x T taps as T 16-byte loads; backward-data, 8 x 8 blocks
enum { kWGather = 0, kWRows = 1, kWBlocks = 2 };

__host__ __device__ constexpr int tile_psu(int NS, int CCG) { return (NS * CCG) | 1; }
// weight records per channel group and per tap: neighbouring groups and taps
// start in other banks, as a wave's writes go to several of them at once
__host__ __device__ constexpr int tile_grec(int OB) { return OB + 1; }
__host__ __device__ constexpr int tile_trec(int CCG, int OB) { return (CCG * tile_grec(OB)) | 1; }

// element e of an array of 16-bit values held in 32-bit words
template <int N>
__device__ __forceinline__ uint32_t pair16(const uint32_t (&d)[N], int e0, int e1) {   // (e0 low, e1 high)
    const uint32_t lo = d[e0 >> 1], hi = d[e1 >> 1];
    const uint32_t sel = ((e0 & 1) ? 0x0302u : 0x0100u) | ((e1 & 1) ? 0x07060000u : 0x05040000u);
    return __builtin_amdgcn_perm(hi, lo, sel);
}

hipError_t launch_tile_bf16(const IgemmArgs& a, hipStream_t s);
hipError_t launch_tile_bf16_bp(const IgemmArgs& a, hipStream_t s);
hipError_t launch_tile_f32(const IgemmArgs& a, hipStream_t s);

// NS: parts per value (1: bf16 tensors, 3: fp32); CCG: 8-channel groups per
// chunk; a wave computes NOBW x NPBW MFMA tiles, WO x WP waves; WM, TT: weight
// staging and its taps (kWRows); WPT, UPT: weight and patch units per thread
// held in registers; BP: the four output phases of a stride-2 backward-data
// together (each tap belongs to one phase; the input patch is shared and the
// two column phases leave as 8-byte stores).  KG: groups of four waves that
// take the channel chunks in turn, each with its own staging buffers, and are
// added at the end: twice the waves per SIMD and half the chain where a layer
// has too few blocks for two workgroups per CU.  SEP: the small part products
// of fp32 have sums of their own (see the plan).
// RAW: the sweep in plain fp32 that follows where the parts do not hold a value
// (see the end); false returned: none is needed.
template <int NS, int CCG, int NOBW, int NPBW, int WO, int WP, int WM, int TT, int WPT, int UPT, bool BP, int KG, bool SEP, bool RAW>
__device__ __forceinline__ bool igemm_tile_sweep(const IgemmArgs& a, unsigned char* smem) {
    static_assert(WO * WP == 4, "four waves");
    static_assert(NS == 1 || WM == kWGather, "fp32 weights are gathered");
    static_assert(!SEP || (NS == 3 && KG == 1 && !RAW), "small part products apart: fp32, one group of waves");
    constexpr int OB = 32 * NOBW * WO, CC = 8 * CCG, NPH = BP ? 4 : 1;
    constexpr int ES = NS == 1 ? 2 : 4;
    constexpr int GW = 16 / ES;             // pixels of a staged 16-byte vector
    constexpr int PSU = tile_psu(NS, CCG);  // records per pixel
    constexpr int GREC = tile_grec(OB), TREC = tile_trec(CCG, OB);

    // pixel blocks round-robin over the XCDs, the output-channel blocks of one
    // pixel block in turn on the same XCD (its patch comes from one L2)
    const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
    const int ob = idx % a.tnob, pbk = (idx / a.tnob) * 8 + xcd;
    if (pbk >= a.tnpb) return false;
    const int per = a.tnub * a.nvb;
    const int z = pbk / per, inb = pbk - z * per;
    const int ub = inb / a.nvb, vb = inb - ub * a.nvb;
    const int tile = z / a.Nn, n = z - tile * a.Nn;
    const int u0 = ub * a.tbu, v0 = vb * a.tbv;
    const int bu = min(a.tbu, a.Uo - u0), bv = a.tbv;   // columns past Vo: computed, not stored
    const int o0 = ob * OB;
    const int T = a.R * a.S;
    const int kg = KG > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kTileThreads) : 0;
    const int tid = threadIdx.x % kTileThreads, wave = tid >> 6, lane = tid & 63;
    const int l32 = lane & 31, hi = lane >> 5;
    const int wo = wave / WP, wp = wave % WP;

    const int plane = a.in_rows * a.in_pitch;
    const char* in = static_cast<const char*>(a.in) + (tile * a.in_tile + int64_t(n) * a.Cin * plane) * ES;
    const __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(in), 0, a.Cin * plane * ES, kTileWord3);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<void*>(a.w), 0, a.wK * a.wC * T * ES, kTileWord3);

    uint4* wl = reinterpret_cast<uint4*>(smem) + kg * a.tgrec;   // [NS][T][CCG][OB], padded
    uint4* pl = wl + NS * T * TREC;               // [PR][ROW][PSU]
    const int WPL = T * TREC;
    int istr = a.istr;
    asm("" : "+s"(istr));   // not loaded again beside LDS writes, which the wait would drain
    const int PG = a.tpg, PR = (bu - 1) * istr + a.Tr;   // 8-pixel groups per row, rows
    const int ROW = PG * GW;
    const int cin0 = v0 * istr + a.base_c, ca = cin0 & ~(GW - 1), sh = cin0 - ca;
    const int row0 = u0 * istr + a.base_r;
    const bool de = istr == 2;   // even and odd columns apart

    // ---- staging units of this thread
    uint32_t poff[UPT];            // patch: byte offset for channel group 0 of a chunk
    int pslot[UPT], pcol[UPT];     // LDS record of pixel 0 (-1: none), its column in the padded row
    const uint32_t pstep = uint32_t(plane) * ES;   // bytes per channel
    auto patch_unit = [&](int e, uint32_t& off, int& slot, int& col) __attribute__((always_inline)) {
        const int cg = e % CCG, rest = e / CCG;
        const int pr = div16(rest, a.tmpg), g = rest - pr * PG;
        const int gr = row0 + pr, gc = ca + g * GW;
        const bool in_lds = pr < PR;
        const bool ok = in_lds & (NS == 1 ? (gr < a.in_rows) & (gc < a.in_pitch)
                                          : (gr >= a.sr0) & (gr < a.sr1) & (gc + GW > a.sc0) & (gc < a.sc1));
        off = ok ? uint32_t(gr * a.in_pitch + gc) * ES + cg * 8 * pstep : kTileOut;
        slot = in_lds ? (pr * ROW + (de ? g * (GW / 2) : g * GW)) * PSU + cg : -1;
        col = gc;
    };
    const int npu = PR * PG * CCG;
#pragma unroll
    for (int q = 0; q < UPT; ++q) patch_unit(tid + q * kTileThreads, poff[q], pslot[q], pcol[q]);

    // weight units: kWGather (tap, group, o) with taps fastest; kWRows (o,
    // group); kWBlocks (group, 8 consecutive (o, tap))
    const int NFG = OB * T / 8;
    const int nwu = WM == kWGather ? T * CCG * OB : WM == kWRows ? OB * CCG : NFG * CCG;
    const uint32_t wstep = uint32_t(a.w_cs) * ES;   // bytes per input channel
    uint32_t woff[WPT];
    int wslot[WPT], wcg[WPT];
    auto w_unit = [&](int e, uint32_t& off, int& slot, int& cg) __attribute__((always_inline)) {
        const bool in_lds = e < nwu;
        if constexpr (WM == kWGather) {
            const int rest = div16(e, a.tmt), t = e - rest * T;
            const int o = a.wmode ? rest % OB : rest / CCG;
            cg = a.wmode ? rest / OB : rest % CCG;
            off = (in_lds & (o0 + o < a.Cout)) ? uint32_t(int((o0 + o) * a.w_os) + t) * ES + cg * 8 * wstep : kTileOut;
            slot = in_lds ? t * TREC + cg * GREC + o : -1;
        } else if constexpr (WM == kWRows) {
            cg = e % CCG;
            const int o = e / CCG;
            off = (in_lds & (o0 + o < a.Cout)) ? uint32_t((o0 + o) * int(a.w_os)) * ES + cg * 8 * wstep : kTileOut;
            slot = in_lds ? cg * GREC + o : -1;
        } else {
            cg = div16(e, a.tmnf);
            const int f = (e - cg * NFG) * 8;
            off = (in_lds & (o0 * T + f < a.Cout * T)) ? uint32_t(o0 * T + f) * ES + cg * 8 * wstep : kTileOut;
            slot = in_lds ? f : -1;
        }
    };
#pragma unroll
    for (int q = 0; q < WPT; ++q) w_unit(tid + q * kTileThreads, woff[q], wslot[q], wcg[q]);

    constexpr int WV = WM == kWRows ? TT : 8;   // vectors (or elements) of a weight unit
    typedef uint32_t u32;
    // channels past Cin: past the sample's end, zero
    auto load_patch = [&](uint4 (&v)[8], uint32_t off, int c0) __attribute__((always_inline)) {
        off += c0 * pstep;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rin, off + j * pstep, 0, 0));
    };
    PartRange range;
    // fp32: the word that says to the whole workgroup that the parts do not hold a
    // value, past the staged records (a static __shared__ word or __syncthreads_or()
    // would come on top of plans that allot the whole LDS); the chunk loop's barriers
    // part this store from any other
    uint32_t* redo = reinterpret_cast<uint32_t*>(smem + a.lds_bytes - kTileRedoBytes);
    if (NS == 3 && !RAW && threadIdx.x == 0) *redo = 0;
    // RAW: the eight channels of a record as fp32 words in its first two
    // parts; the third part's first word marks the patch pixels and the output channels
    // that hold a value the parts do not.
    auto patch_mark = [&](int pixel) __attribute__((always_inline)) {
        return reinterpret_cast<uint32_t*>(pl + pixel * PSU + 2 * CCG);
    };
    auto weight_mark = [&](int o) __attribute__((always_inline)) { return reinterpret_cast<uint32_t*>(wl + 2 * WPL + o); };
    auto put_raw = [](const float (&f)[8], uint4& r0, uint4& r1) __attribute__((always_inline)) {
        uint32_t w[8];
        bool tiny = false;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            w[j] = __builtin_bit_cast(uint32_t, f[j]);
            tiny |= PartRange::tiny(w[j]);
        }
        r0 = uint4{w[0], w[1], w[2], w[3]};
        r1 = uint4{w[4], w[5], w[6], w[7]};
        return tiny;
    };
    auto store_patch = [&](const uint4 (&v)[8], int slot, int col) __attribute__((always_inline)) {
        if (slot < 0) return;
        const int step = PSU, odd = de ? (ROW / 2) * PSU : 0;
        if constexpr (NS == 1) {
            u32 d[8][4];
#pragma unroll
            for (int j = 0; j < 8; ++j) { d[j][0] = v[j].x; d[j][1] = v[j].y; d[j][2] = v[j].z; d[j][3] = v[j].w; }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const u32 sel = (i & 1) ? 0x07060302u : 0x05040100u;
                uint4 r;
                r.x = __builtin_amdgcn_perm(d[1][i / 2], d[0][i / 2], sel);
                r.y = __builtin_amdgcn_perm(d[3][i / 2], d[2][i / 2], sel);
                r.z = __builtin_amdgcn_perm(d[5][i / 2], d[4][i / 2], sel);
                r.w = __builtin_amdgcn_perm(d[7][i / 2], d[6][i / 2], sel);
                pl[slot + (de ? (i / 2) * step + (i & 1) * odd : i * step)] = r;
            }
        } else {
            float f[8][4];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                f[j][0] = __builtin_bit_cast(float, v[j].x); f[j][1] = __builtin_bit_cast(float, v[j].y);
                f[j][2] = __builtin_bit_cast(float, v[j].z); f[j][3] = __builtin_bit_cast(float, v[j].w);
            }
            // columns that feed no stored pixel (the pitch, margins beside an interior) hold anything
            if (col < a.sc0 || col + GW > a.sc1) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (col + i < a.sc0 || col + i >= a.sc1)
#pragma unroll
                        for (int j = 0; j < 8; ++j) f[j][i] = 0.f;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float g[8] = {f[0][i], f[1][i], f[2][i], f[3][i], f[4][i], f[5][i], f[6][i], f[7][i]};
                const int at = slot + (de ? (i / 2) * step + (i & 1) * odd : i * step);
                if constexpr (RAW) {
                    if (put_raw(g, pl[at], pl[at + CCG])) *patch_mark(at / PSU) = 1;
                } else {
                    uint4 p[3];
                    split8(g, p, range);
#pragma unroll
                    for (int s = 0; s < 3; ++s) pl[at + s * CCG] = p[s];
                }
            }
        }
    };
    // channels past Cin lie in the next row of a forward weight tensor: masked
    auto load_w = [&](uint4 (&v)[WV], uint32_t off, int cg, int c0) __attribute__((always_inline)) {
        const int left = a.Cin - c0 - cg * 8;
        off += c0 * wstep;
        if constexpr (WM == kWRows) {
            off |= left > 0 ? 0u : kTileOut;
#pragma unroll
            for (int i = 0; i < TT; ++i)
                v[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rw, off + 16 * i, 0, 0));
        } else if constexpr (WM == kWBlocks) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(
                                                     rw, (off + j * wstep) | (j < left ? 0u : kTileOut), 0, 0));
        }
    };
    auto load_g = [&](u32 (&v)[8], uint32_t off, int cg, int c0) __attribute__((always_inline)) {
        const int left = a.Cin - c0 - cg * 8;
        off += c0 * wstep;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t b = (off + j * wstep) | (j < left ? 0u : kTileOut);
            if constexpr (NS == 1) v[j] = __builtin_amdgcn_raw_buffer_load_b16(rw, b, 0, 0);
            else v[j] = __builtin_amdgcn_raw_buffer_load_b32(rw, b, 0, 0);
        }
    };
    auto store_g = [&](const u32 (&v)[8], int slot) __attribute__((always_inline)) {
        if (slot < 0) return;
        if constexpr (NS == 1) {
            uint4 r;
            r.x = v[0] | (v[1] << 16); r.y = v[2] | (v[3] << 16);
            r.z = v[4] | (v[5] << 16); r.w = v[6] | (v[7] << 16);
            wl[slot] = r;
        } else {
            float f[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) f[j] = __builtin_bit_cast(float, v[j]);
            if constexpr (RAW) {
                if (put_raw(f, wl[slot], wl[slot + WPL])) *weight_mark(slot % TREC % GREC) = 1;
            } else {
                uint4 p[3];
                split8(f, p, range);
#pragma unroll
                for (int s = 0; s < 3; ++s) wl[s * WPL + slot] = p[s];
            }
        }
    };
    // kWBlocks: unit's records held (at) or found on the way; the smallest blocks hold
    // them (72 -> 40 channels on 93x75, three chunks: 17.8 us against 19.2), larger ones
    // have no registers left
    constexpr bool HOLD = WM == kWBlocks && NOBW * NPBW == 1 && !BP && CCG == 4;
    auto w_records = [&](int slot, int cg, int (&at)[8]) __attribute__((always_inline)) {
        int o = div16(slot, a.tmt), t = slot - o * T;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            at[i] = t * TREC + cg * GREC + o;
            const bool wrap = ++t == T;
            t = wrap ? 0 : t;
            o += wrap ? 1 : 0;
        }
    };
    auto store_w = [&](const uint4 (&v)[WV], int slot, int cg, const int* at) __attribute__((always_inline)) {
        if (slot < 0) return;
        if constexpr (WM == kWRows) {
            u32 d[4 * TT];
#pragma unroll
            for (int i = 0; i < TT; ++i) { d[4 * i] = v[i].x; d[4 * i + 1] = v[i].y; d[4 * i + 2] = v[i].z; d[4 * i + 3] = v[i].w; }
#pragma unroll
            for (int t = 0; t < TT; ++t)
                wl[t * TREC + slot] = uint4{pair16(d, t, TT + t), pair16(d, 2 * TT + t, 3 * TT + t),
                                            pair16(d, 4 * TT + t, 5 * TT + t), pair16(d, 6 * TT + t, 7 * TT + t)};
        } else if constexpr (WM == kWBlocks) {
            u32 d[8][4];
#pragma unroll
            for (int j = 0; j < 8; ++j) { d[j][0] = v[j].x; d[j][1] = v[j].y; d[j][2] = v[j].z; d[j][3] = v[j].w; }
            int o = HOLD ? 0 : div16(slot, a.tmt), t = slot - o * T;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const u32 sel = (i & 1) ? 0x07060302u : 0x05040100u;
                uint4 r;
                r.x = __builtin_amdgcn_perm(d[1][i / 2], d[0][i / 2], sel);
                r.y = __builtin_amdgcn_perm(d[3][i / 2], d[2][i / 2], sel);
                r.z = __builtin_amdgcn_perm(d[5][i / 2], d[4][i / 2], sel);
                r.w = __builtin_amdgcn_perm(d[7][i / 2], d[6][i / 2], sel);
                if constexpr (HOLD) {
                    wl[at[i]] = r;
                } else {
                    wl[t * TREC + cg * GREC + o] = r;
                    const bool wrap = ++t == T;
                    t = wrap ? 0 : t;
                    o += wrap ? 1 : 0;
                }
            }
        }
    };

    int wat[HOLD ? WPT : 1][8];
    if constexpr (HOLD) {
#pragma unroll
        for (int q = 0; q < WPT; ++q) w_records(wslot[q], wcg[q], wat[q]);
    }
    uint4 xs[UPT][8];
    uint4 ws[WM == kWGather ? 1 : WPT][WV];
    u32 gs[WM == kWGather ? WPT : 1][8];
    auto load_chunk = [&](int c0) __attribute__((always_inline)) {
        if constexpr (WM == kWGather) {
#pragma unroll
            for (int q = 0; q < WPT; ++q) load_g(gs[q], woff[q], wcg[q], c0);
        } else {
#pragma unroll
            for (int q = 0; q < WPT; ++q) load_w(ws[q], woff[q], wcg[q], c0);
        }
#pragma unroll
        for (int q = 0; q < UPT; ++q) load_patch(xs[q], poff[q], c0);
    };
    auto store_chunk = [&](int c0) __attribute__((always_inline)) {
        if constexpr (!RAW) {   // RAW holds nothing in registers
            if constexpr (WM == kWGather) {
#pragma unroll
                for (int q = 0; q < WPT; ++q) store_g(gs[q], wslot[q]);
            } else {
#pragma unroll
                for (int q = 0; q < WPT; ++q) store_w(ws[q], wslot[q], wcg[q], wat[HOLD ? q : 0]);
            }
#pragma unroll
            for (int q = 0; q < UPT; ++q) store_patch(xs[q], pslot[q], pcol[q]);
        }
        // units beyond the registers' share
        for (int e = tid + (RAW ? 0 : WPT) * kTileThreads; e < nwu; e += kTileThreads) {
            uint32_t off;
            int slot, cg;
            w_unit(e, off, slot, cg);
            if constexpr (WM == kWGather) {
                u32 v[8];
                load_g(v, off, cg, c0);
                store_g(v, slot);
            } else {
                uint4 v[WV];
                load_w(v, off, cg, c0);
                int at[8];
                if constexpr (HOLD) w_records(slot, cg, at);
                store_w(v, slot, cg, at);
            }
        }
        for (int e = tid + (RAW ? 0 : UPT) * kTileThreads; e < npu; e += kTileThreads) {
            uint32_t off;
            int slot, col;
            patch_unit(e, off, slot, col);
            uint4 v[8];
            load_patch(v, off, c0);
            store_patch(v, slot, col);
        }
    };

    floatx16 acc[NPH][NOBW][NPBW];
    floatx16 small[SEP ? NPH : 1][SEP ? NOBW : 1][SEP ? NPBW : 1];   // SEP: sums of the small part products

    // this lane's pixels (past the block's last: a repeat of it, never stored)
    const int np = bu * bv;
    int pix[NPBW];
#pragma unroll
    for (int j = 0; j < NPBW; ++j) {
        const int p = min((wp * NPBW + j) * 32 + l32, np - 1);
        const int ul = div16(p, a.tmbv), vl = p - ul * bv;
        pix[j] = (ul * istr * ROW + (de ? vl : vl * istr)) * PSU;
    }
    const int abase = wo * 32 * NOBW + l32;
    auto tap_b = [&](int tr, int ts) __attribute__((always_inline)) {   // record offset of tap (tr, ts)
        const int c = sh + ts;
        return (tr * ROW + (de ? (c >> 1) + (c & 1) * (ROW / 2) : c)) * PSU;
    };
    // one k-step: records ar of the weights, br of the patch (per lane half)
    auto kstep = [&](int ar, int br, bool zero, int ph) __attribute__((always_inline)) {
        floatx16 (&c)[NOBW][NPBW] = acc[ph];
        constexpr int NR = RAW ? 2 : NS;
        uint4 A[NR][NOBW], B[NR][NPBW];
#pragma unroll
        for (int s = 0; s < NR; ++s) {
#pragma unroll
            for (int i = 0; i < NOBW; ++i) {
                A[s][i] = wl[s * WPL + ar + abase + i * 32];
                if (zero) A[s][i] = uint4{0, 0, 0, 0};
            }
#pragma unroll
            for (int j = 0; j < NPBW; ++j) {
                B[s][j] = pl[br + pix[j] + s * CCG];
                if (zero) B[s][j] = uint4{0, 0, 0, 0};
            }
        }
        if constexpr (RAW) {
            // two channels an instruction, one of each half's group
            static_for<0, 8>([&](auto kc) __attribute__((always_inline)) {
                constexpr int k = decltype(kc)::value;
                auto word = [](const uint4& r) __attribute__((always_inline)) {
                    return __builtin_bit_cast(float, k % 4 == 0 ? r.x : k % 4 == 1 ? r.y : k % 4 == 2 ? r.z : r.w);
                };
#pragma unroll
                for (int i = 0; i < NOBW; ++i)
#pragma unroll
                    for (int j = 0; j < NPBW; ++j)
                        c[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(word(A[k / 4][i]), word(B[k / 4][j]), c[i][j], 0, 0, 0);
            });
        } else {
            constexpr int NP = NS == 1 ? 1 : 6;
            constexpr int pa[6] = {0, 2, 1, 1, 0, 0}, pb[6] = {2, 0, 1, 0, 1, 0};   // small products first
#pragma unroll
            for (int k = 0; k < NP; ++k)
#pragma unroll
                for (int i = 0; i < NOBW; ++i)
#pragma unroll
                    for (int j = 0; j < NPBW; ++j) {
                        floatx16& d = SEP && k + 1 < NP ? small[SEP ? ph : 0][SEP ? i : 0][SEP ? j : 0] : c[i][j];
                        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            __builtin_bit_cast(bf16x8, A[NS == 1 ? 0 : pa[k]][i]),
                            __builtin_bit_cast(bf16x8, B[NS == 1 ? 0 : pb[k]][j]), d, 0, 0, 0);
                    }
        }
    };

    const int cin = a.Tr > 0 ? a.Cin : 0;   // an output phase without taps is zero
    constexpr int STEP = KG * CC;
    // the whole reduction: all channel chunks into acc
    auto sweep = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ph = 0; ph < NPH; ++ph)
#pragma unroll
            for (int i = 0; i < NOBW; ++i)
#pragma unroll
                for (int j = 0; j < NPBW; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        acc[ph][i][j][e] = 0.f;
                        if constexpr (SEP) small[ph][i][j][e] = 0.f;
                    }
        if (!RAW && kg * CC < cin) load_chunk(kg * CC);
        for (int c1 = 0; c1 < cin; c1 += STEP) {
            const int c0 = c1 + kg * CC;
            const bool mine = KG == 1 || c0 < cin;
            if (c1 > 0) __syncthreads();
            if (mine) store_chunk(c0);
            __syncthreads();
            if (!RAW && c0 + STEP < cin) load_chunk(c0 + STEP);
            if (!mine) continue;
            const int ng = min(CCG, (a.Cin - c0 + 7) / 8);   // channel groups of this chunk
#pragma unroll
            for (int ph = 0; ph < NPH; ++ph) {
                const int py = ph >> 1, px = ph & 1;
                const int ntr = BP ? a.bptr[py] : a.Tr, nts = BP ? a.bpts[px] : a.Ts;
                const int dr = BP ? a.bpdr[py] : 0, dcol = BP ? a.bpdc[px] : 0;
                const int r0 = BP ? a.bpr0[py] : a.wr0, rs = BP ? -2 : a.wrstep;
                const int s0 = BP ? a.bps0[px] : a.ws0, ss = BP ? -2 : a.wsstep;
                for (int tr = 0; tr < ntr; ++tr)
                    for (int ts = 0; ts < nts; ++ts) {
                        const int ao = ((r0 + rs * tr) * a.S + s0 + ss * ts) * TREC, bo = tap_b(dr + tr, dcol + ts);
#pragma unroll
                        for (int g = 0; g + 1 < CCG; g += 2)
                            if (g + 1 < ng) kstep(ao + (g + hi) * GREC, bo + g + hi, false, ph);
                    }
                if (ng & 1) {
                    // a last lone group: two taps per k-step, one per half of the lanes
                    const int g = ng - 1, nt = ntr * nts;
                    int tr1 = 0, ts1 = 0;
                    for (int i = 0; i < nt; i += 2) {
                        int tr2 = tr1, ts2 = ts1;
                        if (i + 1 < nt && ++ts2 == nts) { ts2 = 0; ++tr2; }
                        const int tr = hi ? tr2 : tr1, ts = hi ? ts2 : ts1;
                        const int ao = ((r0 + rs * tr) * a.S + s0 + ss * ts) * TREC, bo = tap_b(dr + tr, dcol + ts);
                        kstep(ao + g * GREC, bo + g, (i + 1 >= nt) & hi, ph);
                        tr1 = tr2; ts1 = ts2;
                        if (++ts1 == nts) { ts1 = 0; ++tr1; }
                    }
                }
            }
        }
    };
    // group 1's sums to LDS, added by group 0
    auto join = [&]() __attribute__((always_inline)) {
        if constexpr (KG > 1) {
            typedef float f32x4 __attribute__((ext_vector_type(4)));
            constexpr int NT = NPH * NOBW * NPBW;
            f32x4* red = reinterpret_cast<f32x4*>(smem) + wave * NT * 256 + lane;
            __syncthreads();
            if (kg == 1) {
                static_for<0, NT>([&](auto tc) __attribute__((always_inline)) {
                    constexpr int t = decltype(tc)::value;
                    const floatx16& v = acc[t / (NOBW * NPBW)][t / NPBW % NOBW][t % NPBW];
#pragma unroll
                    for (int q = 0; q < 4; ++q) red[(t * 4 + q) * 64] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
                });
            }
            __syncthreads();
            if (kg == 1) return;
            static_for<0, NT>([&](auto tc) __attribute__((always_inline)) {
                constexpr int t = decltype(tc)::value;
                floatx16& v = acc[t / (NOBW * NPBW)][t / NPBW % NOBW][t % NPBW];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 f = red[(t * 4 + q) * 64];
#pragma unroll
                    for (int j = 0; j < 4; ++j) v[4 * q + j] += f[j];
                }
            });
        }
    };
    if constexpr (RAW) {
        __threadfence();   // the stores of the first sweep are read back below
        for (int e = tid; e < PR * ROW; e += kTileThreads) *patch_mark(e) = 0;
        for (int e = tid; e < OB; e += kTileThreads) *weight_mark(e) = 0;
        __syncthreads();
    }
    sweep();
    if constexpr (SEP) {
#pragma unroll
        for (int ph = 0; ph < NPH; ++ph)
#pragma unroll
            for (int i = 0; i < NOBW; ++i)
#pragma unroll
                for (int j = 0; j < NPBW; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[ph][i][j][e] += small[ph][i][j][e];
    }
    // RAW: the marks of this lane's pixels and output channels, in any group's chunks
    uint32_t marks[RAW ? NPH : 1][RAW ? NPBW : 1] = {}, rows[RAW ? NOBW : 1] = {};
    if constexpr (RAW) {
        __syncthreads();
        for (int k = 0; k < KG; ++k) {
            const uint4* wk = reinterpret_cast<uint4*>(smem) + k * a.tgrec;
            const uint4* pk = wk + NS * T * TREC;
#pragma unroll
            for (int i = 0; i < NOBW; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    rows[i] |= wk[2 * WPL + (wo * NOBW + i) * 32 + 4 * hi + 8 * (e / 4) + e % 4].x ? 1u << e : 0u;
#pragma unroll
            for (int ph = 0; ph < NPH; ++ph) {
                const int py = ph >> 1, px = ph & 1;
                const int ntr = BP ? a.bptr[py] : a.Tr, nts = BP ? a.bpts[px] : a.Ts;
                const int dr = BP ? a.bpdr[py] : 0, dcol = BP ? a.bpdc[px] : 0;
                for (int tr = 0; tr < ntr; ++tr)
                    for (int ts = 0; ts < nts; ++ts)
#pragma unroll
                        for (int j = 0; j < NPBW; ++j) marks[ph][j] |= pk[tap_b(dr + tr, dcol + ts) + pix[j] + 2 * CCG].x;
            }
        }
    }
    join();

    // D of a 32x32 tile: value e of lane l is row 8*(e/4) + 4*(l/32) + e%4
    // (output channel), column l%32 (pixel)
    const int oplane = a.out_rows * a.out_cols;
    float* out = a.out + tile * a.out_tile + int64_t(n) * a.Cout * oplane;
    const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(out, 0, a.Cout * oplane * 4, kTileWord3);
    auto finish = [&](auto ntc) __attribute__((always_inline)) {
        constexpr int AUX = decltype(ntc)::value;
#pragma unroll
        for (int j = 0; j < NPBW; ++j) {
            const int p = (wp * NPBW + j) * 32 + l32;
            const int ul = div16(p, a.tmbv), u = u0 + ul, v = v0 + p - ul * bv;
            const bool live = (p < np) & (v < a.Vo);
#pragma unroll
            for (int i = 0; i < NOBW; ++i) {
                const int ob0 = o0 + (wo * NOBW + i) * 32 + 4 * hi;
                if constexpr (BP) {
#pragma unroll
                    for (int py = 0; py < 2; ++py) {
                        const int orow = 2 * u + py, ocol = 2 * v;
                        const bool ok = live && orow < a.out_rows, both = ocol + 1 < a.out_cols;
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const int o = ob0 + 8 * (e / 4) + e % 4;
                            const uint32_t off = (o * oplane + orow * a.out_cols + ocol) * 4;
                            const float f0 = acc[2 * py][i][j][e], f1 = acc[2 * py + 1][i][j][e];
                            typedef u32 u32x2 __attribute__((ext_vector_type(2)));
                            const u32x2 w2 = {__builtin_bit_cast(u32, f0), __builtin_bit_cast(u32, f1)};
                            __builtin_amdgcn_raw_buffer_store_b64(w2, rout, (ok & both & (o < a.Cout)) ? off : kTileOut, 0, AUX);
                            if (!both & ok & (o < a.Cout)) __builtin_amdgcn_raw_buffer_store_b32(w2[0], rout, off, 0, AUX);
                        }
                    }
                } else {
                    const int orow = u * a.ostr + a.oph_r, ocol = v * a.ostr + a.oph_c;
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int o = ob0 + 8 * (e / 4) + e % 4;
                        const uint32_t off = (o * oplane + orow * a.out_cols + ocol) * 4;
                        const float f = acc[0][i][j][e];
                        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(u32, f), rout,
                                                              (live & (o < a.Cout)) ? off : kTileOut, 0, AUX);
                    }
                }
            }
        }
    };
    if constexpr (!RAW) {
        bool again = false;
        if constexpr (NS == 3) {
            float odd = 0.f;   // NaN where a sum is not finite
            static_for<0, NPH * NOBW * NPBW>([&](auto tc) __attribute__((always_inline)) {
                constexpr int t = decltype(tc)::value;
                float q[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 16; ++e) q[e % 4] = fmaf(acc[t / (NOBW * NPBW)][t / NPBW % NOBW][t % NPBW][e], 0.f, q[e % 4]);
                odd += (q[0] + q[1]) + (q[2] + q[3]);
            });
            if (range.outside() || (kg == 0 && !(odd == 0.f))) *redo = 1;
            __syncthreads();   // before the stores, which it would wait for
            again = *redo;
        }
        if (kg == 0) {
            if (a.nt) finish(std::integral_constant<int, kTileNT>{});
            else finish(std::integral_constant<int, 0>{});
        }
        return again;
    } else {
        if (kg != 0) return false;
#pragma unroll
        for (int ph = 0; ph < NPH; ++ph)
#pragma unroll
            for (int j = 0; j < NPBW; ++j) {
                const int p = (wp * NPBW + j) * 32 + l32;
                const int ul = div16(p, a.tmbv), u = u0 + ul, v = v0 + p - ul * bv;
                const int orow = u * a.ostr + (BP ? ph >> 1 : a.oph_r), ocol = v * a.ostr + (BP ? ph & 1 : a.oph_c);
                if (p >= np || v >= a.Vo || orow >= a.out_rows || ocol >= a.out_cols) continue;
#pragma unroll
                for (int i = 0; i < NOBW; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int o = o0 + (wo * NOBW + i) * 32 + 4 * hi + 8 * (e / 4) + e % 4;
                        if (o >= a.Cout) continue;
                        float* q = out + int64_t(o) * oplane + int64_t(orow) * a.out_cols + ocol;
                        if (marks[ph][j] || (rows[i] >> e & 1) || !isfinite(*q)) *q = acc[ph][i][j][e];
                    }
            }
        return false;
    }
}

// fp32: values the parts cannot hold are noticed while staging (below 2^-110) or by
// what they leave in a sum (too large ones, infinities, NaN).  The block is then
// swept once more on the fp32 instruction, and the outputs that such a value
// reaches, no others, are replaced: an output's bits depend on its own window and
// weights only.  128 -> 128 3x3 on a 64x64 tile: 30 us plain, 73 with one such value
// a tensor, 102 with nothing else; a scalar loop per output took 1,490.
template <int NS, int CCG, int NOBW, int NPBW, int WO, int WP, int WM, int TT, int WPT, int UPT, bool BP, int KG, bool SEP>
__global__ __launch_bounds__(kTileThreads * KG, 2) void igemm_tile_kernel(IgemmArgs) {
    extern __shared__ __align__(16) unsigned char smem[];
    // the arguments where they lie (constant address space: scalar loads); a by-value
    // parameter handed on would be loaded whole at entry
    auto args = __builtin_amdgcn_kernarg_segment_ptr();
    const bool again = igemm_tile_sweep<NS, CCG, NOBW, NPBW, WO, WP, WM, TT, WPT, UPT, BP, KG, SEP, false>(
        *(const IgemmArgs*)args, smem);
    if constexpr (NS == 3) {
        if (!again) return;
        // the arguments read again: kept from the first sweep, the scalars that both
        // derive from them do not fit (159 spilled: the four-phase kernels took 18.6 us
        // instead of 15.6, 32 channels on a 512x512 tile)
        asm volatile("" : "+s"(args));
        igemm_tile_sweep<NS, CCG, NOBW, NPBW, WO, WP, WM, TT, WPT, UPT, BP, KG, false, true>(
            *(const IgemmArgs*)args, smem);
    }
}

template <int NS, int CCG, int NOBW, int NPBW, int WO, int WP, int WM, int TT, int WPT, int UPT, bool BP, int KG = 1, bool SEP = false>
static hipError_t launch_tile(const IgemmArgs& a, hipStream_t s) {
    auto k = igemm_tile_kernel<NS, CCG, NOBW, NPBW, WO, WP, WM, TT, WPT, UPT, BP, KG, SEP>;
    if (a.lds_bytes > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, a.lds_bytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3((a.tnpb + 7) / 8 * 8 * a.tnob), dim3(kTileThreads * KG), a.lds_bytes, s, a);
    return hipGetLastError();
}

}  // namespace dc
