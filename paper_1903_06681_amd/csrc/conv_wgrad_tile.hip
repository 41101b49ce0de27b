// Plan of the blocked weight gradient (conv_wgrad_tile.h).
#include <algorithm>

#include "conv_wgrad_tile.h"

namespace dc {

namespace {

struct Cfg { int id, now, ncw, wo, wc, wt, wk, tw; };
#define X(id, now, ncw, wo, wc, wt, wk, tw) {id, now, ncw, wo, wc, wt, wk, tw},
const Cfg kCfgs[] = {DC_WT_CONFIGS(X)};
#undef X

}  // namespace

bool wgrad_tile_plan(int dtype, int ntiles, int N, int C, int K, int R, int S, int st, int Hot, int Wot,
                     int base_c, int dy_off, WgradTile* t) {
    const int NS = dtype == 1 ? 1 : 3, ES = dtype == 1 ? 2 : 4, GW = 16 / ES;
    const int T = R * S;
    if (base_c < 0) return false;
    // byte offsets within a sample are 32-bit, with room for a block's channels past the
    // end; the padded x tile has at most these rows and columns
    const int64_t xr = int64_t(Hot) * st + R + st + 2 * int64_t(dy_off), xc = int64_t(Wot) * st + S + st + 2 * int64_t(dy_off) + 16;
    const int64_t dr = Hot + 2 * int64_t(dy_off), dcols = Wot + 2 * int64_t(dy_off) + 16;
    if ((C + 128) * xr * xc * ES >= int64_t(kWtOut) || (K + 128) * dr * dcols * ES >= int64_t(kWtOut)) return false;
    const bool c32 = C <= 32, k32 = K <= 32, c64 = C <= 64, k64 = K <= 64;
    // blocks of filters x channels: the smallest that the layer fills
    int id;
    if (T == 1) id = NS == 3 ? 7 : k64 && c64 ? 7 : k64 ? 8 : c64 ? 9 : 6;
    else if (T <= 9) id = k32 && c32 ? 3 : k32 ? 2 : c32 ? 1 : 0;
    else if (T <= 28) id = NS == 1 && !k32 && !c32 ? 10 : 4;
    else id = 5;
    const Cfg& f = kCfgs[id];
    const int P = wt_pixels(NS, id);
    const int OBK = 32 * f.now * f.wo, CBK = 32 * f.ncw * f.wc, NOB = OBK / 32, NCB = CBK / 32;
    const int extra = NS == 3 ? kWtRedoBytes : 0;
    const int limit = device_lds_limit() - extra;
    const int nws = f.wo * f.wc * f.wt, nbw = f.tw * f.now * f.ncw;
    const int64_t red = f.wk > 1 ? int64_t(f.wk / 2) * nws * nbw * 4096 : 0;
    if (red > limit) return false;
    const int64_t images = int64_t(ntiles) * N;
    double best = 0;
    bool found = false;
    const int nv0 = (Wot + P - 1) / P, nv1 = std::min((Wot + 7) / 8, nv0 + 31);
    for (int nv = nv0; nv <= nv1; ++nv) {
        int bv = (Wot + nv - 1) / nv;
        if (nv > 1) bv = (bv + 7) / 8 * 8;
        if (bv > P) continue;
        const int nvb = (Wot + bv - 1) / bv;
        for (int bu = std::min(Hot, P / bv); bu >= 1; --bu) {
            const int nub = (Hot + bu - 1) / bu;
            if ((Hot + nub - 1) / nub != bu) continue;   // balanced rows only
            const int pg = (base_c % GW + (bv - 1) * st + S + GW - 1) / GW, dg = (dy_off % GW + bv + GW - 1) / GW;
            const int pr = (bu - 1) * st + R;
            const int64_t lds = int64_t(NS) * (NOB * (P + 2) + NCB * (int64_t(pr) * pg * GW + 1)) * 64;
            if (lds > limit) continue;
            const int nbuf = lds * 2 <= limit ? 2 : 1;
            const int64_t npb = images * nub * nvb;
            if (npb > (int64_t(1) << 30)) continue;
            // cycles of a block: matrix work of its k-steps on four SIMDs, staging, a barrier
            const int ks = (bu * bv + 15) / 16;
            const double mf = double((ks + f.wk - 1) / f.wk) * std::min(T, f.tw) * f.now * f.ncw * (NS == 3 ? 6 : 1) * 64.0;
            const double stage = (double(pr) * pg * GW * CBK + double(bu) * dg * GW * OBK) * (NS == 3 ? 0.09 : 0.035);
            // staging units past one per thread are loaded without being requested ahead
            const int units = ((bu * dg * OBK / 8 + 63) & ~63) + pr * pg * CBK / 8;
            const double late = NS == 3 && units > kWtThreads ? 1500.0 : 0.0;
            const double cost = double(npb) * (mf + stage + late + (nbuf == 2 ? 400.0 : 900.0));
            if (!found || cost < best) {
                found = true;
                best = cost;
                t->tbu = bu; t->tbv = bv; t->tnub = nub; t->nqb = nvb; t->tpg = pg; t->tdg = dg;
                t->tnpb = int(npb); t->tnbuf = nbuf;
                t->lds_bytes = int(std::max(lds * nbuf, red)) + extra;
            }
        }
    }
    if (!found) return false;
    t->tcfg = id;
    t->now = f.now; t->ncw = f.ncw; t->wo = f.wo; t->wc = f.wc;
    t->gy = (T + f.wt * f.tw - 1) / (f.wt * f.tw);
    t->gz = ((K + OBK - 1) / OBK) * ((C + CBK - 1) / CBK);
    t->F = int64_t(t->gz) * T * f.wo * f.wc * f.now * f.ncw * 1024;
    // Chunks: at most one workgroup per CU, and 64 MiB of partials (what the
    // allocation-free entry point holds) where one chunk's stay below it; more of them shorten the walk over the
    // pixel blocks (matrix work and about 1 us of barriers and exposed latency
    // each), fewer move less: each chunk writes and reads F floats, taken
    // at 10 TB/s (most of them stay in the caches).  Above eight a whole number per XCD, so that the blocks of one chunk
    // share an L2.
    const int64_t most = std::max<int64_t>(1, std::min<int64_t>({std::max(1, device_cu_count() / (t->gy * t->gz)),
                                                                  (int64_t(64) << 20) / (t->F * 4), t->tnpb}));
    const double block_us = best / t->tnpb / 2.2e3 + 1.0, chunk_us = double(t->F) * 8.0 / 1e7;
    int64_t nch = 1;
    double cheapest = 0;
    for (int64_t n = 1;; n = std::min(most, n < 8 ? n + 1 : n + 8)) {
        const double us = double((t->tnpb + n - 1) / n) * block_us + double(n) * chunk_us;
        if (n == 1 || us < cheapest) { cheapest = us; nch = n; }
        if (n == most) break;
    }
    t->tbpc = int((t->tnpb + nch - 1) / nch);
    t->nchunks = (t->tnpb + t->tbpc - 1) / t->tbpc;
    auto magic = [](int d) { return d > 1 ? uint32_t((uint64_t(1) << 32) / uint32_t(d) + 1) : 0u; };
    t->tmpg = magic(t->tpg); t->tmdg = magic(t->tdg); t->tmbv = magic(t->tbv);
    return true;
}

// dw = (accumulate ? dw : 0) + the sum of the chunks' partials: chunk group g
// (of G) adds chunks g, g + G, ... in order, then groups 0 .. G - 1.  A
// workgroup takes 256 consecutive floats of the partials, a quarter of one
// 32 x 32 block, so that the block's place is scalar arithmetic and each
// thread moves four filters' values with 16-byte loads.  Bound: HBM (the
// partials); where the quarters leave CUs idle the round trips of one thread,
// hence sixteen groups from 32 chunks on (us: 256 chunks of 36 quarters, fp32
// 32 -> 32 stride 2 on a 512x512 tile, 8.9 with four groups, 6.7 with sixteen;
// 64 chunks of 576 quarters 8.4 and 11.7).
template <int G>
__global__ __launch_bounds__(64 * G) void wgrad_tile_reduce_kernel(WgradArgs a) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    __shared__ f32x4 red[G][64];
    const int q = blockIdx.x & 3, blk = blockIdx.x >> 2, lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int nb = a.tnow * a.tncw, T = a.R * a.S;
    const int b = blk % nb, w = blk / nb, wc = w % a.twc, wo = w / a.twc % a.two, zz = w / (a.twc * a.two);
    const int tap = zz % T, bz = zz / T;
    const int cbk = 32 * a.tncw * a.twc, ncsb = (a.C + cbk - 1) / cbk;
    const int o0 = (((bz / ncsb) * a.two + wo) * a.tnow + b / a.tncw % a.tnow) * 32 + 8 * q;
    const int c0 = (((bz % ncsb) * a.twc + wc) * a.tncw + b % a.tncw) * 32;
    if (o0 >= a.K || c0 >= a.C) return;
    const f32x4* src = reinterpret_cast<const f32x4*>(a.part) + int64_t(blockIdx.x) * 64 + lane;
    const int64_t step = a.F / 4;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    int c = g;
    for (; c + 3 * G < a.nchunks; c += 4 * G) {   // four loads in flight, added in chunk order
        f32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = src[(c + G * j) * step];
#pragma unroll
        for (int j = 0; j < 4; ++j) sum += v[j];
    }
    for (; c < a.nchunks; c += G) sum += src[c * step];
    red[g][lane] = sum;
    __syncthreads();
    if (g != 0) return;
    f32x4 total = red[0][lane];
#pragma unroll
    for (int k = 1; k < G; ++k) total += red[k][lane];
    const int o = o0 + 4 * (lane >> 5), ci = c0 + (lane & 31);
    if (ci >= a.C) return;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (o + j < a.K) {
            float* d = a.dw + (int64_t(o + j) * a.C + ci) * T + tap;
            *d = a.accumulate ? *d + total[j] : total[j];
        }
}

hipError_t launch_wgrad_tile(const WgradArgs& a, int dtype, hipStream_t s) {
    hipError_t e = dtype == 1 ? launch_wgrad_tile_bf16(a, s) : launch_wgrad_tile_f32(a, s);
    if (e != hipSuccess) return e;
    const dim3 grid(unsigned(a.F / 256));
    if (a.nchunks >= 32 && a.F <= 65536) hipLaunchKernelGGL(wgrad_tile_reduce_kernel<16>, grid, dim3(64 * 16), 0, s, a);
    else hipLaunchKernelGGL(wgrad_tile_reduce_kernel<4>, grid, dim3(64 * 4), 0, s, a);
    return hipGetLastError();
}

}  // namespace dc
