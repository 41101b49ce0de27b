// Weight gradient of layers of any channel count, filter, image size and
// stride on gfx950 matrix cores (Eq. (2) of Sec. II-A restricted to the tile).
//
//   dw[o][ci, tap] = sum over output pixels of dy[o][pixel] * x[ci][pixel shifted by tap]
//
// Work split.  A workgroup of eight waves owns OBK filters x CBK channels at
// WT x TW taps and walks a chunk of pixel blocks (tbu x tbv output pixels of
// one image, at most P).  A block's dy pixels and x patch are staged once in
// LDS; each wave keeps its 32 x 32 blocks at TW taps in accumulators.  WK
// groups of waves take the block's 16-pixel k-steps in turn and are added in
// LDS at the end: the partials that leave the workgroup, a fixed 36 KB per
// wave with nine taps, are what large layers would otherwise spend most of
// their time on.
//
// LDS layout.  The reduction runs over pixels, so a lane needs eight
// consecutive pixels of one channel, at any shift.  Both operands lie
// pixel-major, 32 channels (64 bytes) a record, and are read with the
// transposing read of gfx950 (ds_read_b64_tr_b16: 16 lanes read 4 pixels x 16
// channels and each gets 4 pixels of its channel).  Every lane names its own
// pixel, so a tap's shift, a row end inside a k-step and the column stride are
// only addresses: blocks are flattened and narrow images waste nothing.  At
// column stride 2 even and odd columns of the patch lie apart, which keeps
// the four pixels of a read in different banks.
//
// Pixels past the block's last (and outside the tile) hold zero dy and read x
// from a zero record, so that no value outside the sum meets the matrix unit.
//
// fp32 layers use three bf16 parts per value and six part products, as the
// blocked convolution does (conv_igemm_tile.h; error against 64 bits 0.75 of the
// row kernel's over 44 layers of mesh models, one 2 % above it); chunks whose values the parts
// cannot hold are swept once more on the fp32 instruction.
//
// Bound: staging (two channels of 16-byte loads, transposes and LDS writes per
// block) and one barrier a block; matrix work is about a quarter.  Measured
// against the row kernels, us a pass with the reduction: bf16 256 -> 256 3x3
// stride 2 on 32 images of 28x28 823 -> 36; 64 -> 64 stride 2 on 112x112, N=2:
// 75 -> 16; 1x1 stride 2 256 -> 512 on 28x28, N=16: 422 -> 21; fp32 32 -> 32
// stride 2 on a 512x512 tile 105 -> 34; fp32 128 -> 128 on a 64x64 tile 43 -> 28.
#pragma once

#include <hip/hip_runtime.h>

#include "bf16util.h"
#include "kernels.h"

namespace dc {

static constexpr int kWtThreads = 512;
static constexpr int kWtWord3 = 0x00020000;          // buffer resource word 3 (gfx9 family: raw access)
static constexpr uint32_t kWtOut = 0x80000000u;      // byte offset past every buffer here: loads 0
static constexpr int kWtRedoBytes = 16;              // fp32: LDS of the redo word, past everything else

template <int NS, int NOW, int NCW, int WO, int WC, int WT, int WK, int TW, int P, int UPT>
__global__ __launch_bounds__(kWtThreads, 2) void wgrad_tile_kernel(WgradArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    static_assert(WO * WC * WT * WK == 8, "eight waves");
    constexpr int ES = NS == 1 ? 2 : 4, GW = 16 / ES;
    constexpr int OBK = 32 * NOW * WO, CBK = 32 * NCW * WC;
    constexpr int NOB = OBK / 32, NCB = CBK / 32;
    constexpr int DPIX = P + 2;            // dy records: P pixels, one nobody reads, one of zeros
    constexpr int KPW = (P / 16 + WK - 1) / WK;
    typedef uint32_t u32;
    typedef float f32x4 __attribute__((ext_vector_type(4)));

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wk = wave / (WO * WC * WT), wsub = wave % (WO * WC * WT);
    const int wt = wsub / (WO * WC), wo = (wsub / WC) % WO, wc = wsub % WC;
    const int T = a.R * a.S, st = a.istr;
    const int ncsb = (a.C + CBK - 1) / CBK;
    const int o0 = (blockIdx.z / ncsb) * OBK, c0 = (blockIdx.z % ncsb) * CBK;
    const int tap0 = (blockIdx.y * WT + wt) * TW;

    const int xplane = a.x_rows * a.x_pitch, dplane = (a.Hot + 2 * a.dy_off) * a.dy_pitch;
    const int PG = a.tpg, DG = a.tdg, ROW = PG * GW, PR = (a.tbu - 1) * st + a.R;
    const int XPIX = PR * ROW + 1;         // odd: the 32-channel planes start in other banks
    const bool de = st == 2;
    // staging buffer: dy records, then x records, 64 bytes each
    const int buf_bytes = (NS * (NOB * DPIX + NCB * XPIX)) * 64;
    const int XO = NS * NOB * DPIX * 64;
    const int shx = a.base_c % GW, shd = a.dy_off % GW;
    // x rows and columns up to here are read by the sums; fp32: what lies outside is
    // staged as zero, as the contents of a cell may choose the arithmetic of its chunk
    const int xr1 = a.base_r + (a.Hot - 1) * st + a.R, xc1 = a.base_c + (a.Wot - 1) * st + a.S;

    // ---- staging units: dy first (rounded up to whole waves), then x
    const int ndu = (a.tbu * DG * (OBK / 8) + 63) & ~63;
    const int nxu = PR * PG * (CBK / 8);
    struct Unit { u32 off; int rec; int col; int row; };   // byte offset, LDS record, first column / pixel, row
    auto make_unit = [&](int e, Unit& u) __attribute__((always_inline)) {
        const bool isd = __builtin_amdgcn_readfirstlane(e) < ndu;
        if (isd) {
            const int cg = e % (OBK / 8), rest = e / (OBK / 8);
            const int r = div16(rest, a.tmdg), g = rest - r * DG;
            const bool ok = r < a.tbu;
            u.row = ok ? r : 1 << 20;
            u.col = g * GW - shd;                          // output column of the vector's first element
            u.off = (u32((a.dy_off + r) * a.dy_pitch + a.dy_off - shd + g * GW) +
                     u32(o0 + cg * 8) * dplane) * ES;
            u.rec = ((cg / 4) * DPIX) * 4 + cg % 4;
        } else {
            const int f = e - ndu, cg = f % (CBK / 8), rest = f / (CBK / 8);
            const int r = div16(rest, a.tmpg), g = rest - r * PG;
            const bool ok = r < PR;
            u.row = ok ? r : 1 << 20;
            u.col = a.base_c - shx + g * GW;               // tile column, without the block's
            u.off = (u32((a.base_r + r) * a.x_pitch + u.col) + u32(c0 + cg * 8) * xplane) * ES;
            u.rec = ((cg / 4) * XPIX + r * ROW + (de ? g * (GW / 2) : g * GW)) * 4 + cg % 4;
        }
    };
    Unit un[UPT];
#pragma unroll
    for (int q = 0; q < UPT; ++q) make_unit(tid + q * kWtThreads, un[q]);

    // ---- blocks of this chunk
    const int b0 = blockIdx.x * a.tbpc, b1 = min(b0 + a.tbpc, a.tnpb);
    const int per = a.tnub * a.nqb;
    struct Block { const char* x; const char* dy; int u0, v0; };
    auto block = [&](int b) __attribute__((always_inline)) {
        const int z = b / per, inb = b - z * per, ub = inb / a.nqb, vb = inb - ub * a.nqb;
        const int tile = z / a.Nn, n = z - tile * a.Nn;
        Block k;
        k.x = static_cast<const char*>(a.x) + (tile * a.x_tile + int64_t(n) * a.C * xplane) * ES;
        k.dy = static_cast<const char*>(a.dy) + (tile * a.dy_tile + int64_t(n) * a.K * dplane) * ES;
        k.u0 = ub * a.tbu;
        k.v0 = vb * a.tbv;
        return k;
    };
    auto load_unit = [&](uint4 (&v)[8], const Unit& u, int e, const Block& k) __attribute__((always_inline)) {
        const bool isd = __builtin_amdgcn_readfirstlane(e) < ndu;
        const char* base = isd ? k.dy : k.x;
        const u32 step = u32(isd ? dplane : xplane) * ES;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(base), 0, int(step) * (isd ? a.K : a.C), kWtWord3);
        const int row = u.row + (isd ? k.u0 : a.base_r + k.u0 * st);
        const int col = u.col + (isd ? a.dy_off + k.v0 : k.v0 * st);
        const int rows = isd ? a.Hot : NS == 1 ? a.x_rows : xr1, cols = isd ? a.dy_pitch : NS == 1 ? a.x_pitch : xc1;
        const bool ok = (row < rows) & (col < cols);
        const u32 at = u.off + (isd ? u32(k.u0 * a.dy_pitch + k.v0) : u32((k.u0 * a.x_pitch + k.v0) * st)) * ES;
        const u32 off = ok ? at : kWtOut;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, off + j * step, 0, 0));
    };
    PartRange range;
    // rawc: plain fp32, the eight channels of a record as fp32 words in its first two parts
    auto store_unit = [&](auto rawc, const uint4 (&v)[8], const Unit& u, int e, const Block& k, unsigned char* buf)
        __attribute__((always_inline)) {
        if (u.row >= 1 << 20) return;
        const bool isd = __builtin_amdgcn_readfirstlane(e) < ndu;
        uint4* l = reinterpret_cast<uint4*>(buf + (isd ? 0 : XO)) + u.rec;
        const int splane = (isd ? NOB * DPIX : NCB * XPIX) * 4;   // records between parts
        auto put = [&](int i, int at, bool live) __attribute__((always_inline)) {
            auto word = [&](int j, int w) __attribute__((always_inline)) {
                return w == 0 ? v[j].x : w == 1 ? v[j].y : w == 2 ? v[j].z : v[j].w;
            };
            if constexpr (NS == 1) {
                const u32 sel = (i & 1) ? 0x07060302u : 0x05040100u;
                uint4 r;
                r.x = __builtin_amdgcn_perm(word(1, i / 2), word(0, i / 2), sel);
                r.y = __builtin_amdgcn_perm(word(3, i / 2), word(2, i / 2), sel);
                r.z = __builtin_amdgcn_perm(word(5, i / 2), word(4, i / 2), sel);
                r.w = __builtin_amdgcn_perm(word(7, i / 2), word(6, i / 2), sel);
                r.x = live ? r.x : 0; r.y = live ? r.y : 0; r.z = live ? r.z : 0; r.w = live ? r.w : 0;
                l[at] = r;
            } else {
                float f[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) f[j] = live ? __builtin_bit_cast(float, word(j, i)) : 0.f;
                if constexpr (decltype(rawc)::value) {
                    l[at] = __builtin_bit_cast(uint4, f32x4{f[0], f[1], f[2], f[3]});
                    l[at + splane] = __builtin_bit_cast(uint4, f32x4{f[4], f[5], f[6], f[7]});
                } else {
                    uint4 p[3];
                    split8(f, p, range);
#pragma unroll
                    for (int s = 0; s < 3; ++s) l[at + s * splane] = p[s];
                }
            }
        };
        if (isd) {
            // elements outside the tile's interior are zero, those outside the block's
            // columns go to the record nobody reads
            const int end = a.Wot - k.v0 - u.col, row = u.row * a.tbv;
#pragma unroll
            for (int i = 0; i < GW; ++i) {
                const int vl = u.col + i;
                const bool in = (vl >= 0) & (vl < a.tbv);
                put(i, (in ? row + vl : P) * 4, in & (i < end));
            }
        } else {
            // the row's first and last vectors: the pitch, and in fp32 what no sum reads, hold anything
            const int col = u.col + k.v0 * st, c1 = NS == 1 ? a.x_cols : xc1;
            if ((NS == 1 || col >= a.base_c) && c1 - col >= GW) {
#pragma unroll
                for (int i = 0; i < GW; ++i) put(i, (de ? (i / 2) + (i & 1) * (ROW / 2) : i) * 4, true);
            } else {
#pragma unroll
                for (int i = 0; i < GW; ++i)
                    put(i, (de ? (i / 2) + (i & 1) * (ROW / 2) : i) * 4, (NS == 1 || col + i >= a.base_c) & (i < c1 - col));
            }
        }
    };
    const int nu = ndu + nxu;
    uint4 xs[UPT][8];
    auto load_block = [&](const Block& k) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < UPT; ++q) load_unit(xs[q], un[q], tid + q * kWtThreads, k);
    };
    auto store_block = [&](auto rawc, const Block& k, unsigned char* buf) __attribute__((always_inline)) {
        constexpr bool RAW = decltype(rawc)::value;   // holds nothing in registers
        if constexpr (!RAW) {
#pragma unroll
            for (int q = 0; q < UPT; ++q) store_unit(rawc, xs[q], un[q], tid + q * kWtThreads, k, buf);
        }
        for (int e = tid + (RAW ? 0 : UPT) * kWtThreads; e < ((nu + 63) & ~63); e += kWtThreads) {
            Unit u;
            make_unit(e, u);
            uint4 v[8];
            load_unit(v, u, e, k);
            store_unit(rawc, v, u, e, k, buf);
        }
    };

    // ---- this lane's read positions: lane reads channels 4 (l%4) + 16 ((l/16)%2) .. + 3
    // of pixel 8 (l/32) + (l%16)/4 (+ 4 for the second read) of a k-step
    const int chb = (lane & 3) * 8 + ((lane >> 4) & 1) * 32;
    const int pl0 = 8 * (lane >> 5) + ((lane & 15) >> 2);
    int xoff[KPW][2];
#pragma unroll
    for (int q = 0; q < KPW; ++q)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int p = min((q * WK + wk) * 16 + pl0 + 4 * h, a.tbu * a.tbv - 1);
            const int ul = div16(p, a.tmbv), vl = p - ul * a.tbv;
            xoff[q][h] = (ul * st * ROW + (de ? vl : vl * st)) * 64 + chb;
        }
    int toff[TW];   // byte offset of a tap (uniform)
#pragma unroll
    for (int i = 0; i < TW; ++i) {
        const int t = min(tap0 + i, T - 1), r = t / a.S, s = t - r * a.S, c = shx + s;
        toff[i] = (r * ROW + (de ? (c >> 1) + (c & 1) * (ROW / 2) : c)) * 64;
    }
    floatx16 acc[TW][NOW][NCW];

    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4* lds4;
    const u32 lds0 = u32(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)smem));
    auto frag = [&](u32 p0, u32 p1) __attribute__((always_inline)) {
        const s16x4 f0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(uintptr_t)p0);
        const s16x4 f1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(uintptr_t)p1);
        return __builtin_bit_cast(bf16x8, __builtin_shufflevector(f0, f1, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    constexpr int NP = NS == 1 ? 1 : 6;
    constexpr int pa[6] = {0, 2, 1, 1, 0, 0}, pb[6] = {2, 0, 1, 0, 1, 0};   // small products first
    auto compute = [&](u32 base, int bu, int bv) __attribute__((always_inline)) {
        const int np = bu * a.tbv;
        const u32 zero = base + (DPIX - 1) * 64 + chb;     // the zero record of dy plane 0
#pragma unroll
        for (int q = 0; q < KPW; ++q) {
            const int kk = q * WK + wk;
            if (kk * 16 >= np) continue;
            const bool whole = (kk * 16 + 16 <= np) & (bv == a.tbv);
            bool in0 = true, in1 = true;
            if (!whole) {
                const int p0 = kk * 16 + pl0, p1 = p0 + 4;
                in0 = (p0 < np) & (p0 - div16(p0, a.tmbv) * a.tbv < bv);
                in1 = (p1 < np) & (p1 - div16(p1, a.tmbv) * a.tbv < bv);
            }
            bf16x8 A[NS][NOW];
#pragma unroll
            for (int s = 0; s < NS; ++s)
#pragma unroll
                for (int o = 0; o < NOW; ++o) {
                    const u32 d = base + ((s * NOB + wo * NOW + o) * DPIX + kk * 16 + pl0) * 64 + chb;
                    A[s][o] = frag(d, d + 4 * 64);
                }
            auto read_b = [&](bf16x8 (&B)[NS][NCW], int off) __attribute__((always_inline)) {
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int c = 0; c < NCW; ++c) {
                        const u32 x = base + XO + ((s * NCB + wc * NCW + c) * XPIX) * 64 + off;
                        const u32 x0 = x + xoff[q][0], x1 = x + xoff[q][1];
                        B[s][c] = frag(in0 ? x0 : zero, in1 ? x1 : zero);
                    }
            };
            // operands are read AH taps ahead of their products (the barriers keep the
            // compiler from moving the reads back; past the last tap: a repeat, not stored)
            constexpr int AH = NS == 1 && NCW == 1 ? 2 : 1, NB = AH + 1;
            bf16x8 B[NB][NS][NCW];
#pragma unroll
            for (int i = 0; i < AH && i < TW; ++i) read_b(B[i], toff[i]);
            static_for<0, TW>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                if constexpr (i + AH < TW) read_b(B[(i + AH) % NB], toff[i + AH]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < NP; ++k)
#pragma unroll
                    for (int o = 0; o < NOW; ++o)
#pragma unroll
                        for (int c = 0; c < NCW; ++c)
                            acc[i][o][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                A[NS == 1 ? 0 : pa[k]][o], B[i % NB][NS == 1 ? 0 : pb[k]][c], acc[i][o][c], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    };

    // the same sums on the fp32 instruction, two pixels each: a lane's half takes pixels
    // 8 (l/32) .. + 7 of a k-step, its filter and channel are l%32 of their blocks
    auto compute_raw = [&](unsigned char* buf, int bu, int bv) __attribute__((always_inline)) {
        const int np = bu * a.tbv, l32 = lane & 31;
        const int word = (l32 / 8) * 16 + (l32 & 3) * 4, part = (l32 >> 2) & 1;
        auto at = [&](int off) __attribute__((always_inline)) { return *reinterpret_cast<const float*>(buf + off + word); };
        for (int k = wk * 16; k < np; k += WK * 16)
            for (int m = 0; m < 8; ++m) {
                const int p = k + 8 * (lane >> 5) + m, ul = div16(p, a.tmbv), vl = p - ul * a.tbv;
                const bool in = (p < np) & (vl < bv);
                const int px = (ul * st * ROW + (de ? vl : vl * st)) * 64;
                float A[NOW];
#pragma unroll
                for (int o = 0; o < NOW; ++o) A[o] = at(((part * NOB + wo * NOW + o) * DPIX + p) * 64);
                static_for<0, TW>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
#pragma unroll
                    for (int c = 0; c < NCW; ++c) {
                        const float B = at(in ? XO + (part * NCB + wc * NCW + c) * XPIX * 64 + px + toff[i] : (DPIX - 1) * 64);
#pragma unroll
                        for (int o = 0; o < NOW; ++o)
                            acc[i][o][c] = __builtin_amdgcn_mfma_f32_32x32x2f32(A[o], B, acc[i][o][c], 0, 0, 0);
                    }
                });
            }
    };

    // fp32: the word that says to the whole workgroup that the parts do not hold a
    // value, past the staged records and the sums (a static __shared__ word or
    // __syncthreads_or() would come on top of plans that allot the whole LDS)
    u32* redo_word = reinterpret_cast<u32*>(smem + a.lds_bytes - kWtRedoBytes);
    if (NS == 3 && tid == 0) *redo_word = 0;
    // all pixel blocks of the chunk into acc
    auto sweep = [&](auto rawc) __attribute__((always_inline)) {
        constexpr bool RAW = decltype(rawc)::value;
        static_for<0, TW * NOW * NCW>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i / (NOW * NCW)][i / NCW % NOW][i % NCW][e] = 0.f;
        });
        // dy records past the block's pixels are never staged: zero them once (and the
        // zero record) in every buffer
        for (int e = tid; e < a.tnbuf * NS * NOB * DPIX * 4; e += kWtThreads) {
            const int per_buf = NS * NOB * DPIX * 4, b = e / per_buf, f = e - b * per_buf;
            *(reinterpret_cast<uint4*>(smem + b * buf_bytes) + f) = uint4{0, 0, 0, 0};
        }
        if (b0 >= b1) return;
        if constexpr (RAW) {
            for (int b = b0; b < b1; ++b) {
                const Block k = block(b);
                __syncthreads();
                store_block(rawc, k, smem);
                __syncthreads();
                compute_raw(smem, min(a.tbu, a.Hot - k.u0), min(a.tbv, a.Wot - k.v0));
            }
        } else {
            Block cur = block(b0);
            load_block(cur);
            __syncthreads();
            store_block(rawc, cur, smem);
            Block nxt = b0 + 1 < b1 ? block(b0 + 1) : cur;
            if (b0 + 1 < b1) load_block(nxt);
            __syncthreads();
            for (int b = b0; b < b1; ++b) {
                const int cb = a.tnbuf == 2 ? (b - b0) & 1 : 0;
                compute(lds0 + cb * buf_bytes, min(a.tbu, a.Hot - cur.u0), min(a.tbv, a.Wot - cur.v0));
                if (b + 1 == b1) break;
                if (a.tnbuf == 1) __syncthreads();
                store_block(rawc, nxt, smem + (a.tnbuf == 2 ? (cb ^ 1) * buf_bytes : 0));
                cur = nxt;
                if (b + 2 < b1) {
                    nxt = block(b + 2);
                    load_block(nxt);
                }
                __syncthreads();
            }
        }
    };

    // ---- the wave groups' sums, added pairwise in LDS in a fixed order
    constexpr int NBW = TW * NOW * NCW, NWS = WO * WC * WT;
    f32x4* red = reinterpret_cast<f32x4*>(smem);
    auto join = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int half = WK / 2; half >= 1; half /= 2) {
            __syncthreads();
            if (wk >= half && wk < 2 * half) {
                f32x4* d = red + (((wk - half) * NWS + wsub) * NBW) * 256 + lane;
                static_for<0, NBW>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    const floatx16& v = acc[i / (NOW * NCW)][i / NCW % NOW][i % NCW];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        d[(i * 4 + q) * 64] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
                });
            }
            __syncthreads();
            if (wk < half) {
                const f32x4* d = red + ((wk * NWS + wsub) * NBW) * 256 + lane;
                static_for<0, NBW>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    floatx16& v = acc[i / (NOW * NCW)][i / NCW % NOW][i % NCW];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 f = d[(i * 4 + q) * 64];
#pragma unroll
                        for (int j = 0; j < 4; ++j) v[4 * q + j] += f[j];
                    }
                });
            }
        }
    };
    sweep(std::false_type{});
    join();
    if constexpr (NS == 3) {
        // Values the parts cannot hold: below 2^-110 noticed while staging, and too large
        // ones, infinities and NaN by what they leave in a sum.  The chunk is then swept
        // once more on the fp32 instruction (128 -> 128 3x3 on a 64x64 tile: 30 us plain, 44
        // with one such value, 49 with nothing else; a scalar loop per sum took 1,110).
        float odd = 0.f;   // NaN where a sum is not finite
        static_for<0, NBW>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
#pragma unroll
            for (int e = 0; e < 16; ++e) odd = fmaf(acc[i / (NOW * NCW)][i / NCW % NOW][i % NCW][e], 0.f, odd);
        });
        if (range.outside() || (wk == 0 && !(odd == 0.f))) *redo_word = 1;
        __syncthreads();
        if (*redo_word) {
            sweep(std::true_type{});
            join();
        }
    }
    // partial: [chunk][gz][tap][wave of the tap][o block][c block][4][64 lanes][4], the
    // filter's taps only; value j of lane l in quarter q is row 8 q + 4 (l/32) + j
    // (filter), column l%32 (channel)
    if (wk > 0) return;
    constexpr int NB = NOW * NCW;
    float* part = a.part + int64_t(blockIdx.x) * a.F +
                  ((int64_t(blockIdx.z) * T + tap0) * (WO * WC) + wo * WC + wc) * NB * 1024;
    static_for<0, NBW>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        if (tap0 + i / NB >= T) return;
        const floatx16& v = acc[i / NB][i / NCW % NOW][i % NCW];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            reinterpret_cast<f32x4*>(part)[(i / NB * (WO * WC) * NB + i % NB) * 256 + q * 64 + lane] =
                f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
    });
}

template <int NS, int NOW, int NCW, int WO, int WC, int WT, int WK, int TW, int P, int UPT>
static hipError_t launch_wgrad_tile(const WgradArgs& a, hipStream_t s) {
    auto k = wgrad_tile_kernel<NS, NOW, NCW, WO, WC, WT, WK, TW, P, UPT>;
    if (a.lds_bytes > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, a.lds_bytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3(a.nchunks, a.gy, a.gz), dim3(kWtThreads), a.lds_bytes, s, a);
    return hipGetLastError();
}

// Instantiations: id, 32x32 blocks per wave (filters, channels), wave grid
// (filters, channels, taps, k-groups), taps per wave.
#define DC_WT_CONFIGS(X) \
    X(0, 1, 1, 2, 2, 2, 1, 5)  /* 64 x 64, ten taps */ \
    X(1, 1, 1, 2, 1, 2, 2, 5)  /* 64 x 32 */ \
    X(2, 1, 1, 1, 2, 2, 2, 5)  /* 32 x 64 */ \
    X(3, 1, 1, 1, 1, 2, 4, 5)  /* 32 x 32 */ \
    X(4, 1, 1, 1, 1, 4, 2, 7)  /* 32 x 32, 28 taps */ \
    X(5, 1, 1, 1, 1, 8, 1, 7)  /* 32 x 32, 56 taps */ \
    X(6, 2, 2, 2, 2, 1, 2, 1)  /* 128 x 128, one tap */ \
    X(7, 2, 2, 1, 1, 1, 8, 1)  /* 64 x 64, one tap */ \
    X(8, 2, 2, 1, 2, 1, 4, 1)  /* 64 x 128, one tap */ \
    X(9, 2, 2, 2, 1, 1, 4, 1)  /* 128 x 64, one tap */ \
    X(10, 1, 1, 2, 2, 2, 1, 7) /* 64 x 64, fourteen taps */

// Pixels of a block: 128, in fp32 64 where the operands are wider than 32 (three
// parts of two buffers of 128 do not fit the LDS).
constexpr int wt_pixels(int NS, int id) { return NS == 1 || id == 3 ? 128 : 64; }

}  // namespace dc
