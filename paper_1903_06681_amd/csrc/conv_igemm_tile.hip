// Plan of the blocked implicit GEMM (conv_igemm_tile.h).
#include <algorithm>

#include "conv_igemm_tile.h"

namespace dc {

namespace {

struct Cfg { int id, OB, PT, NOBW, NPBW; };

}  // namespace

bool igemm_tile_plan(IgemmArgs& a, int dtype) {
    if (a.frame || a.bp == 1) return false;
    const int NS = dtype == 1 ? 1 : 3, ES = dtype == 1 ? 2 : 4, GW = 16 / ES;
    const int T = a.R * a.S;
    // byte offsets of a sample, the weights and an output sample are 32-bit
    // with room for a last chunk's channels past the end
    const int64_t cap = kTileOut;
    if (int64_t(a.Cin + 64) * a.in_rows * a.in_pitch * ES >= cap || int64_t(a.wK + 64) * (a.wC + 64) * T * ES >= cap ||
        int64_t(a.Cout + 128) * a.out_rows * a.out_cols * 4 >= cap)
        return false;
    if (a.in_pitch % GW != 0 || a.base_r < 0 || a.base_c < 0) return false;
    // channels per chunk: as many as leave two workgroups of LDS per CU
    int ccg;
    if (NS == 1) ccg = T == 1 ? 8 : T <= 12 ? 4 : 2;
    else ccg = T == 1 ? 4 : 2;
    int wm = kWGather;
    if (NS == 1) {
        if (a.wmode == 0 && (T == 9 || T == 1) && a.Cin % 8 == 0) wm = kWRows;
        else if (a.wmode == 1 && int64_t(a.Cout) * T % 8 == 0) wm = kWBlocks;
        if (wm != kWRows && a.Cin <= 16) ccg = 2;
    }
    const int extra = NS == 3 ? kTileRedoBytes : 0;
    const int limit = device_lds_limit(), cus = device_cu_count();
    static const Cfg plain_bf16[] = {{0, 64, 256, 2, 2}, {1, 64, 128, 2, 1}, {2, 64, 64, 1, 1}, {3, 32, 256, 1, 2}, {4, 128, 128, 2, 2}};
    static const Cfg plain_f32[] = {{1, 64, 128, 2, 1}, {2, 64, 64, 1, 1}, {3, 32, 256, 1, 2}, {5, 32, 128, 1, 1}};
    static const Cfg bp_bf16[] = {{1, 64, 128, 2, 1}, {2, 64, 64, 1, 1}, {5, 32, 128, 1, 1}};
    static const Cfg bp_f32[] = {{2, 64, 64, 1, 1}, {5, 32, 128, 1, 1}};
    const Cfg* cfgs = a.bp ? (NS == 1 ? bp_bf16 : bp_f32) : (NS == 1 ? plain_bf16 : plain_f32);
    const int nc = a.bp ? (NS == 1 ? 3 : 2) : (NS == 1 ? 5 : 4);
    // The block shape with the least estimated time: rounds of workgroups x
    // (chunks x the larger of the matrix work of the workgroups on a CU and
    // one workgroup's matrix work plus staging).
    const int64_t images = int64_t(a.ntiles) * a.Nn;
    const int nchunk = (a.Cin + 8 * ccg - 1) / (8 * ccg);
    const int groups = (a.Cin + 7) / 8;
    const int taps = a.bp ? T : a.Tr * a.Ts;
    const double ksteps = double(taps) * groups / 2.0 / nchunk;   // per chunk
    // Two groups of waves on the chunks where one tile's nominal 64 x 128 blocks
    // leave CUs without a second workgroup and there are chunks to share (fp32
    // 128 -> 128 on a 64x64 tile: 42 -> 29 us; bf16 256 -> 256 stride 2 on 28x28,
    // N=32: 34 -> 25).  The four phases of a stride-2 backward-data make four times
    // the outputs of a block: at 256 blocks one group is faster (31 against 40).
    // The rule reads one tile's sizes only: the order of the sums does not depend
    // on how many tiles a launch has.
    const int64_t nominal = int64_t(a.Nn) * ((int64_t(a.Uo) * a.Vo + 127) / 128) * ((a.Cout + 63) / 64);
    const bool pair = nominal <= (a.bp ? cus / 2 : cus) && nchunk >= 4 &&
                      (NS == 3 ? ccg == 2 : ccg == 4 && (wm == kWBlocks || (wm == kWRows && T == 9)));
    // fp32 on few channels: a group of eight that is mostly empty makes six additions
    // of one or a few products, each rounded at the size of the sum, where the fp32
    // instruction makes one for every two channels.  The five small part products of
    // each k-step then have sums of their own, added at the end.  Error of y against 64
    // bits (fp32 instruction, one sum, two sums): 3 -> 16 channels 3x3 stride 2 9.6e-8,
    // 1.2e-7, 3.9e-8; 17 -> 9 2.2e-7, 2.4e-7, 7.6e-8, in the same time.  From 19 channels
    // on, whole groups make fewer additions than the fp32 instruction (32 channels 3.0e-7,
    // 2.5e-7), and 64 x 128 blocks, whose registers do not hold second sums, are worth having.
    a.tsep = NS == 3 && !a.bp && a.Cin <= 18;
    double best = 0;
    bool found = false;
    for (int kg = pair ? 2 : 1; kg >= 1 && !found; --kg)
    for (int c = 0; c < nc; ++c) {
        const Cfg& f = cfgs[c];
        if (a.tsep && f.id == 1) continue;
        if (kg == 2 && NS == 1 && !a.bp && (f.id == 0 || f.id == 4)) continue;
        if (wm == kWGather && NS == 1 && !a.bp && (f.id == 0 || f.id == 4)) continue;
        const int nob = (a.Cout + f.OB - 1) / f.OB;
        const int nv0 = (a.Vo + f.PT - 1) / f.PT, nv1 = std::min((a.Vo + 7) / 8, nv0 + 31);
        for (int nv = nv0; nv <= nv1; ++nv) {
            int bv = (a.Vo + nv - 1) / nv;
            if (nv > 1) bv = (bv + GW - 1) / GW * GW;
            if (bv > f.PT) continue;
            const int nvb = (a.Vo + bv - 1) / bv;
            int bu = std::min(a.Uo, f.PT / bv);
            const int nub = (a.Uo + bu - 1) / bu;
            bu = (a.Uo + nub - 1) / nub;
            // columns a block reads, from an aligned start
            const int shm = (bv * a.istr) % GW == 0 || nvb == 1 ? a.base_c % GW : GW - 1;
            const int pg = (shm + (bv - 1) * a.istr + std::max(a.Ts, 1) + GW - 1) / GW;
            const int pr = (bu - 1) * a.istr + a.Tr;
            const int64_t grec = int64_t(NS) * T * tile_trec(ccg, f.OB) + int64_t(pr) * pg * GW * tile_psu(NS, ccg);
            const int64_t sums = kg == 2 ? int64_t(a.bp ? 4 : 1) * f.NOBW * f.NPBW * 4 * 4096 : 0;
            const int64_t lds = std::max(grec * 16 * kg, sums) + extra;
            if (lds > limit) continue;
            const int occ = lds * 2 <= limit ? 2 : 1;
            const int64_t npb = images * nub * nvb;
            if ((npb + 8) * nob > (int64_t(1) << 30)) continue;
            const int64_t nwg = npb * nob;
            const double mf = ksteps * f.NOBW * f.NPBW * (NS == 3 ? 6 : 1) * 32.0;
            const double stage = 700.0 + double(grec) / 3.0 * (NS == 3 ? 1.5 : 1.0);
            const int64_t slots = int64_t(cus) * occ;
            const int k = kg * int(std::min<int64_t>(occ, (nwg + cus - 1) / cus));
            const double per = double((nchunk + kg - 1) / kg) * std::max(k * mf, mf + stage) + 4000.0 + (kg - 1) * 1500.0;
            const double cost = per * double((nwg + slots - 1) / slots);
            if (!found || cost < best) {
                found = true;
                best = cost;
                a.tcfg = f.id; a.OB = f.OB; a.tnob = nob;
                a.tbu = bu; a.tbv = bv; a.tnub = nub; a.nvb = nvb;
                a.tpg = pg; a.tnpb = int(npb);
                a.lds_bytes = int(lds);
                a.tkg = kg; a.tgrec = int(grec);
                // whole 64-byte sectors of a large output bypass the caches (64 -> 256 1x1
                // on 56x56, N=32, 103 MB: 39 -> 25 us; with blocks of 196 pixels, whose
                // sectors are shared, on 28x28: 14 -> 24).  With a reader right after, a
                // conversion to bf16, 60 -> 65 us there and 15.8 -> 16.7 on 26 MB; fp32 layers,
                // slower to write, gain with it too (32 channels stride 2 input gradient on a
                // 512x512 tile 26.6 -> 26.4, alone 18.1 -> 16.7).
                const bool rows = a.out_cols % 16 == 0 && bv % 16 == 0;
                const bool flat = !a.bp && a.ostr == 1 && nvb == 1 && (int64_t(a.out_rows) * a.out_cols) % 16 == 0 &&
                                  int64_t(bu) * bv % 16 == 0;
                a.nt = (rows || flat) && int64_t(a.Nn) * a.Cout * a.out_rows * a.out_cols * 4 >= (int64_t(8) << 20);
            }
        }
    }
    if (!found) return false;
    a.twm = wm; a.tccg = ccg;
    a.sr0 = std::max(a.base_r, a.own);
    a.sr1 = std::min(a.base_r + (a.Uo - 1) * a.istr + a.Tr, a.in_rows - a.own);
    a.sc0 = std::max(a.base_c, a.own);
    a.sc1 = std::min(a.base_c + (a.Vo - 1) * a.istr + a.Ts, a.in_cols - a.own);
    auto magic = [](int d) { return d > 1 ? uint32_t((uint64_t(1) << 32) / uint32_t(d) + 1) : 0u; };
    a.tmt = magic(T); a.tmpg = magic(a.tpg); a.tmbv = magic(a.tbv); a.tmnf = magic(a.OB * T / 8);
    a.kind = 5;
    return true;
}

hipError_t launch_igemm_tile(const IgemmArgs& a, int dtype, hipStream_t s) {
    if (dtype != 1) return launch_tile_f32(a, s);
    return a.bp ? launch_tile_bf16_bp(a, s) : launch_tile_bf16(a, s);
}

}  // namespace dc
