// Plan of the rolling-row kernel (conv_igemm_roll.h) and its 3x3 instantiations
// with system-scope stores.
#include "conv_igemm_roll.h"

namespace dc {

hipError_t launch_roll3_nt(const IgemmArgs& a, hipStream_t s);
hipError_t launch_roll5(const IgemmArgs& a, hipStream_t s);

bool igemm_roll_plan(IgemmArgs& a) {
    if (a.bp || a.istr != 1 || a.ostr != 1 || a.oph_r != 0 || a.oph_c != 0) return false;
    if (a.Cin % 16 != 0 || a.Cout % 32 != 0 || a.Vo % kRStrip != 0) return false;
    if (a.base_c % 8 != 0 || a.in_pitch % 8 != 0 || a.Tr != a.R || a.Ts != a.S) return false;
    const int NOB = a.Cout % 64 == 0 ? 2 : 1, CG = a.Cin / 16;
    if (!roll_shape(NOB, a.Tr, a.Ts, CG)) return false;
    if (a.wmode == 0 && !(a.wr0 == 0 && a.wrstep == 1 && a.ws0 == 0 && a.wsstep == 1)) return false;
    if (a.wmode == 1 && !(a.wr0 == a.R - 1 && a.wrstep == -1 && a.ws0 == a.S - 1 && a.wsstep == -1))
        return false;
    const int T = a.R * a.S;
    if (a.wmode == 0 && (int64_t(a.Cin) * T) % 8 != 0) return false;
    if (a.wmode == 1 && (int64_t(a.Cout) * T) % 8 != 0) return false;
    // 32-bit buffer offsets
    const int64_t in_plane = int64_t(a.in_rows) * a.in_pitch, oplane = int64_t(a.out_rows) * a.out_cols;
    if (int64_t(a.Cin) * in_plane * 2 >= (int64_t(1) << 31) || 64 * oplane * 4 >= (int64_t(1) << 31)) return false;
    if (a.out_rows < a.Uo || a.out_cols < a.Vo) return false;
    const int lds = roll_lds(NOB, a.Tr, a.Ts, CG);
    if (lds > device_lds_limit()) return false;
    // equal segments of at least TR rows, about 256 workgroups
    a.nvb = a.Vo / kRStrip;
    const int strips = a.ntiles * a.Nn * a.nvb * (a.Cout / (32 * NOB));
    int best = 0;
    for (int rps = a.Tr; rps <= a.Uo; ++rps) {
        if (a.Uo % rps != 0) continue;
        best = rps;
        if (int64_t(strips) * (a.Uo / rps) <= 256) break;
    }
    if (best == 0) return false;
    a.rows_per_seg = best;
    a.nseg = a.Uo / best;
    a.OB = 32 * NOB;
    // Non-temporal stores of large outputs: with inputs and outputs that change from
    // call to call (c5a, 67 MB) the forward takes 26 us against 32, backward-data 24
    // against 29; on 34 MB (c5b, 5x5) system scope is 0.5 us faster.  Part of that
    // moves to a reader right after, which finds nothing in the caches: with a
    // conversion of the output to bf16 behind the call, 48 us against 46 forward and
    // 48 against 45 backward-data; on 134 MB (N = 8) 43 against 56 alone, 89 against 83.
    a.nt = NOB == 2 && int64_t(a.Nn) * a.Cout * oplane * 4 >= (int64_t(48) << 20);
    a.wvec = 1;
    a.phase = 0;
    a.lds_bytes = lds;
    a.kind = 3;
    return true;
}

hipError_t launch_igemm_roll(const IgemmArgs& a, hipStream_t s) {
    const int CG = a.Cin / 16;
    if (a.OB == 64 && a.Tr == 3 && a.Ts == 3 && CG == 4 && a.rows_per_seg >= 3) {
        if (a.nt) return launch_roll3_nt(a, s);
        switch (a.rows_per_seg % 3) {
            case 0: return launch_roll<2, 3, 3, 4, 0, false>(a, s);
            case 1: return launch_roll<2, 3, 3, 4, 1, false>(a, s);
            default: return launch_roll<2, 3, 3, 4, 2, false>(a, s);
        }
    }
    if (a.OB == 32 && a.Tr == 5 && a.Ts == 5 && CG == 2 && a.rows_per_seg >= 5) return launch_roll5(a, s);
    return hipErrorInvalidValue;
}

}  // namespace dc
