// Selection policies over the feasible set F = {(leaf, E) : the leaf's system
// holds at the bound machine and at E, and an instance of its program exists}.
//
// CASE: the paper fixes the leaf for given parameters by the case discussion
// and leaves the program parameters to auto-tuning (Section 1); here they are
// chosen by an analytic estimate of the launch time:
//   tiles     = ceil(M / tile_m) * ceil(N / tile_n) * shares of K
//   rounds    : the busiest compute unit's tiles, by as many as it holds at a
//               time (LDS, registers, threads, workgroup slots)
//   per round = K steps * max(workgroups * 2 * tile_m * tile_n * bk / rate,
//                             step latency) + opening and closing
//               rate: per-CU throughput of the program's inner loop (matrix
//               cores; or VALU multiply-adds limited by the LDS words read per
//               multiply-add), the share of it that a tile sustains falling
//               with the words moved per flop, 1/tile_m + 1/tile_n, and with
//               too few wavefronts to hide latencies; step latency: one
//               global-load round trip plus the barriers of a K step
//   traffic   = bytes the tiles read (each tile reads its A and B panels) over
//               an on-chip cache bandwidth, and the operands' bytes over HBM
//   estimate  = max(rounds, traffic) + a fixed launch cost
// The constants were fitted to event timings of these kernels on gfx950; the
// estimate only has to rank candidates.
// EXHAUSTIVE: every candidate is launched and timed with HIP events on the
// device (back-to-back launches, mean), the least CASE estimate first; a
// candidate whose first three launches are already 1.5x slower than the best
// so far is not timed further, nor one whose single warm-up launch takes over
// a millisecond and twice the best.  The fastest is kept (cached per shape).
#include "select.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <stdexcept>

namespace pk {

namespace {
constexpr double kHbmBytesPerSecond = 8e12;

int elem_bytes(int dtype) { return dtype == PK_BF16 ? 2 : 4; }

}  // namespace

double product_rate(const pk_machine &m, const KernelEntry &e, int dtype) {
    const int threads = e.threads;
    const int wave = m.wave > 0 ? m.wave : 64;
    const double lanes = (double)threads / (double)(wave * ((threads + wave - 1) / wave));
    // MFMA: float32 256, bfloat16 2048; int32 on the int8 matrix cores 8192
    // int8 operations per clock, ten int8 products per int32 one
    if (e.family == PK_FAMILY_MFMA) return dtype == PK_BF16 ? 2048.0 : dtype == PK_I32 ? 819.2 : 256.0;
    // VALU: 64 lanes x 4 SIMDs / 4 cycles = 64 multiply-adds per clock for
    // float32; int32 multiply-adds run at half of that (measured).  The tiled kernel
    // also reads 1 + s LDS words per s multiply-adds, which caps it near 24
    // multiply-adds per clock, rising slowly with s; the direct kernel is
    // bound by global/L1 reads (about one multiply-add per clock).
    // int32 (fitted on the timings of every feasible candidate of 200 random
    // int32 shapes, 140 to fit and 60 to check): the tiled kernel's relative
    // rates 0.85, 0.9, 0.5, 0.7 for s = 1, 2, 4, 8 of the 32 multiply-adds
    // per clock; the 2-D micro-tile program (four k of A and s columns of B
    // per LDS read) up to 1.1 times that, or about 36 LDS words per clock.
    const double s = std::max(1, e.s);
    double mads = dtype == PK_I32 ? 32.0 : 64.0;
    if (e.family == PK_FAMILY_VALU2) {
        // 2-D micro-tiles: (s + sy) / (s sy) LDS words per multiply-add
        // against the LDS's words per clock, up to the ALU rate
        const double sy = std::max(1, e.sy);
        if (dtype == PK_I32) return 2.0 * lanes * std::min(mads * 1.1, 36.0 * s * sy / (s + sy));
        return 2.0 * lanes * std::min(mads, 24.0 * s * sy / (s + sy));
    }
    if (e.variant & PK_VALU_NOLDS)
        mads = 1.0;
    else if (dtype == PK_I32)
        mads *= e.s <= 1 ? 0.85 : e.s == 2 ? 0.9 : e.s <= 4 ? 0.5 : 0.70;
    else
        mads = std::min(mads, 24.0 * std::pow(s / (1.0 + s), 0.25));
    return 2.0 * mads * lanes;
}

double streaming_seconds(const pk_machine &m, const KernelEntry &e, double bytes, int64_t tiles,
                         double inflight_bytes_per_tile, double segment_bytes) {
    const int64_t ncu = std::max<int32_t>(m.cu_count, 1);
    const int64_t bpc = blocks_per_cu(m, e);
    tiles = std::max<int64_t>(tiles, 1);
    const int64_t per_cu = (tiles + ncu - 1) / ncu;  // tiles of the busiest compute unit
    const int64_t active = std::min(ncu, tiles);
    const double imbalance = (double)(per_cu * ncu) / (double)tiles;
    const double resident = (double)std::min(bpc, per_cu);
    const double inflight = std::min(1.0, resident * inflight_bytes_per_tile / 65536.0);
    // a wavefront's access is 64 lanes x 4 bytes: runs along a row shorter
    // than 256 bytes split it over several rows (transposition of order 2^14:
    // the 128-byte runs of 32-wide tiles 4.4 TB/s, the 256-byte ones 4.9)
    const double seg = std::min(1.0, segment_bytes / 256.0);
    // one compute unit alone draws about 64 GB/s; all of them, 8 TB/s
    const double bw = std::min(8e12, 64e9 * (double)active) * 0.85 * std::max(inflight * seg, 1e-3);
    const double rounds = (double)((per_cu + bpc - 1) / bpc);
    return bytes * (tiles >= ncu ? imbalance : 1.0) / bw + 0.5e-6 * rounds + 3e-6;
}

namespace {

// The MFMA programs' estimate, by element type.  Fitted to the timings of
// every candidate of 260 (float32, bfloat16) or 130 (int32) products of 64 to
// 8192 along each dimension, packed and padded rows, three sets of operands in
// turn, so that the least estimate is the fastest program or close to it:
// half of the products to fit, half to check.  The choice's mean time over the
// fastest's, before and with these: float32 1.049 and 1.021, bfloat16 1.040
// and 1.014, int32 1.186 and 1.039.  The float32 and bfloat16 kernels for
// unaligned rows got faster since (several K steps in registers); with the
// present ones, on 100 float32, 80 int32 and 80 bfloat16 packed products drawn
// anew, whose rows are mostly unaligned: 1.024, 1.020 and 1.025.
struct MfmaFit {
    double waves;          // wavefronts a SIMD needs to hide latencies (fourth root below)
    double eff, edge;      // share of the peak rate eff / (1 + edge (1 / tile_m + 1 / tile_n))
    double lat1, lat2;     // least seconds of a K step, single-stage and two-stage programs
    double narrow, nlat;   // factors on both where rows are not aligned
    double shallow;        // arithmetic of wide wavefronts that have registers for two
                           // buffers of K steps only (max_depth): bfloat16 of order 4096,
                           // 151 us on 256 x 128 tiles and 124 on 128 x 256
    double open;           // seconds a tile opens and closes in
    double panels, hbm;    // bytes per second of the tiles' panels, and of the operands once
    double split, adds;    // a split product's second launch (2 us of the device, but 4 of
                           // the caller's thread: float32 of order 256, 9.4 us a call on
                           // one launch, 12.9 split); atomic additions per second
    double launch;         // seconds
};
constexpr MfmaFit kFit[3] = {
    /* float32  */ {1.16, 1.03, 2.28, 2.0e-6, 0.228e-6, 1.28, 3.33, 1.0, 1.17e-6, 9.67e12, 1.79e12, 4e-6, 4.18e11, 2.4e-6},
    /* int32    */ {5.76, 1.12, 6.9, 0.324e-6, 0.174e-6, 1.1, 1.0, 1.0, 1.95e-6, 25e12, 0.82e12, 5.5e-6, 0.55e11, 2.18e-6},
    /* bfloat16 */ {2.1, 0.938, 14.5, 0.05e-6, 0.156e-6, 2.29, 2.92, 1.19, 2.01e-6, 11.8e12, 4.2e12, 4e-6, 4.49e11, 1.84e-6},
};

// The VALU programs' estimate, float32 and int32.  Products with a dimension
// below 64 decide between them and the MFMA programs, and were not among those
// that the constants above were fitted to: a K step that few workgroups share
// takes the latency of its loads and of its barriers, and the operands' bytes
// cost what they cost the MFMA programs (kFit's hbm).  The smallest products
// are a launch and a store: on the device 2.6 to 3 us with a VALU program and 4.2
// with an MFMA one, whose launch and open kFit counts as 3.6 to 4.1.  Fitted to half of
// 570 int32 and 470 float32 products of 1 to 8192 along each dimension, two
// thirds of them with one below 64, and of 160 each of up to 50 MFLOP; mean
// time of the choice over the fastest program's on all of the former and all
// of the latter: int32 1.04 and 1.02, float32 1.04 and 1.02.  Before the
// operands' bytes and the latency counted: 1.22 and 1.10 on the former (int32
// 37 x 4544 x 3168: 317 us chosen, 50 now; float32 7692 x 6808 x 18: 206 and
// 49); with constants of the former alone: 1.08 and 1.23 on the latter (int32
// 617 x 26 x 50, float32 63 x 527 x 3).
struct ValuFit {
    double launch;              // seconds
    double latency, latency_k;  // least seconds of a K step, and per k of a tiled program's
    double barriers;            // seconds of a step's barriers per resident workgroup
};
constexpr ValuFit kValuFit[2] = {
    /* float32 */ {3.15e-6, 0.045e-6, 0.0048e-6, 0.55e-6},
    /* int32   */ {2.9e-6, 0.085e-6, 0.0013e-6, 0.37e-6},
};

double fourth(double x) { return x * x * x * x; }
double fourth_root(double x) { return std::sqrt(std::sqrt(x)); }

// The launch's seconds under an MFMA program of which a compute unit holds
// `resident` workgroups: the busiest unit runs its tiles in rounds of the
// resident ones, a K step of a round taking the larger of the tiles'
// arithmetic and one step's latency; beside that the panels' and the operands'
// bytes, the largest of the three deciding (all three soft, as fourth powers'
// sums).
double estimate_mfma(const pk_machine &m, const KernelEntry &e, int64_t resident, double prate, int dtype, int64_t M,
                     int64_t N, int64_t K, bool wide, int ks) {
    const MfmaFit &f = kFit[dtype];
    const double clock = (m.clock_khz > 0 ? m.clock_khz : 2400000) * 1e3;
    const int64_t ncu = std::max<int32_t>(m.cu_count, 1);
    const int wave = m.wave > 0 ? m.wave : 64;
    const int64_t tiles = std::max<int64_t>(((M + e.tile_m - 1) / e.tile_m) * ((N + e.tile_n - 1) / e.tile_n), 1) * ks;
    const int64_t per_cu = (tiles + ncu - 1) / ncu;
    const int64_t res = std::min(resident, per_cu), full = per_cu / res, rest = per_cu % res;
    const int bk = e.bk > 0 ? e.bk : 1;
    const double ksteps = std::ceil((double)((std::max<int64_t>(K, 1) + bk - 1) / bk) / ks);
    const bool shallow = wide && dtype == PK_BF16 && pkk::max_depth(false, e.bm, e.bn, e.wm, e.wn) < 3;
    const double flops = 2.0 * e.tile_m * e.tile_n * bk * (wide ? 1.0 : f.narrow) * (shallow ? f.shallow : 1.0);
    const double rate = prate * clock * f.eff / (1.0 + f.edge * (1.0 / e.tile_m + 1.0 / e.tile_n));
    const double latency = ((e.variant & PK_MFMA_SINGLE) ? f.lat1 : f.lat2) * (wide ? 1.0 : f.nlat) *
                           (dtype == PK_I32 ? bk / 32.0 : 1.0);  // (int32: the digits of every 32 k)
    auto round = [&](int64_t r) {
        if (r <= 0) return 0.0;
        const double waves = (double)r * ((e.threads + wave - 1) / wave) / 4.0;
        const double work = (double)r * flops / (rate * fourth_root(std::min(1.0, waves / f.waves)));
        return ksteps * fourth_root(fourth(work) + fourth(latency)) + f.open;
    };
    const double compute = (double)full * round(res) + round(rest);
    const double es = elem_bytes(dtype);
    // each workgroup reads its A and B panels over its share of K
    const double panels = es * (double)tiles * std::ceil((double)K / ks) * (e.tile_m + e.tile_n) / f.panels;
    const double hbm = (es * ((double)M * K + (double)K * N) + 4.0 * (double)M * N) / f.hbm;
    // shares of K: clearing C (a second launch) and one atomic addition per
    // output and share
    const double split = ks > 1 ? f.split + 4.0 * (double)M * N / 5e12 + (double)ks * M * N / f.adds : 0.0;
    return fourth_root(fourth(compute) + fourth(panels) + fourth(hbm)) + split + f.launch;
}

// estimate_seconds with the program's residency and rate given (the bound
// table holds them per point)
double estimate_program(const pk_machine &m, const KernelEntry &e, int64_t resident, double prate, int dtype,
                        int64_t M, int64_t N, int64_t K, bool wide, int ks) {
    ks = std::max(ks, 1);
    if (e.family == PK_FAMILY_MFMA) return estimate_mfma(m, e, resident, prate, dtype, M, N, K, wide, ks);
    // VALU programs.  Per compute unit: the busiest one holds
    // ceil(tiles / NCU) tiles, `res` of them resident at once; each K step of
    // a round costs the larger of the resident tiles' arithmetic at the unit's
    // rate and one step's latency, and two barriers per resident workgroup;
    // beside that the tiles' and the operands' bytes.
    // The rate falls when few wavefronts share a SIMD to hide LDS and memory
    // latency (full at about three per SIMD), and where workgroups have fewer
    // than 256 work-items, in proportion.
    const double clock = (m.clock_khz > 0 ? m.clock_khz : 2400000) * 1e3;
    const int64_t ncu = std::max<int32_t>(m.cu_count, 1);
    const int wave = m.wave > 0 ? m.wave : 64;
    const int64_t tm = (M + e.tile_m - 1) / e.tile_m, tn = (N + e.tile_n - 1) / e.tile_n;
    const int64_t tiles = std::max<int64_t>(tm * tn, 1);
    const int64_t per_cu = (tiles + ncu - 1) / ncu;
    const int64_t res = std::min(resident, per_cu);
    const int64_t rounds = (per_cu + res - 1) / res;
    const int bk = e.bk > 0 ? e.bk : 1;
    const double ksteps = (double)((std::max<int64_t>(K, 1) + bk - 1) / bk);
    const double flops_step = 2.0 * e.tile_m * e.tile_n * bk;
    const double waves_per_simd = (double)res * ((e.threads + wave - 1) / wave) / 4.0;
    const double occupancy = waves_per_simd >= 3.0 ? 1.0 : fourth_root(waves_per_simd / 3.0);
    const double rate = prate * clock * std::min(1.0, e.threads / 256.0) * occupancy;
    const ValuFit &f = kValuFit[dtype];
    const double latency = f.latency + ((e.variant & PK_VALU_NOLDS) ? 0.0 : f.latency_k * bk);
    const double overhead = f.barriers * (double)res;
    const double compute = (double)rounds * ksteps * (std::max((double)res * flops_step / rate, latency) + overhead);
    const double es = elem_bytes(dtype);
    const double tile_bytes = es * (double)tiles * (double)K * (e.tile_m + e.tile_n);
    const double hbm = (es * ((double)M * K + (double)K * N) + 4.0 * (double)M * N) / kFit[dtype].hbm;
    return std::max(compute, std::max(tile_bytes / kHbmBytesPerSecond, hbm)) + f.launch;
}

}  // namespace

// The workgroups the estimate takes a compute unit to hold.  MFMA programs:
// what gfx950's registers (512 a lane and SIMD), LDS and wave slots admit; the
// runtime's register figure, which the case table takes as reported, may be
// half of that.  Others: the model's count, to which their estimate is fitted.
int64_t estimate_residency(const pk_machine &m, const KernelEntry &e) {
    if (e.family != PK_FAMILY_MFMA || std::strncmp(m.arch, "gfx950", 6) != 0) return blocks_per_cu(m, e);
    pk_machine hw = m;
    hw.regs_cu = std::max<int64_t>(m.regs_cu, 131072);
    return blocks_per_cu(hw, e);
}

double estimate_seconds(const pk_machine &m, const KernelEntry &e, int dtype, int64_t M, int64_t N, int64_t K,
                        bool wide, int ks) {
    return estimate_program(m, e, estimate_residency(m, e), product_rate(m, e, dtype), dtype, M, N, K, wide, ks);
}

double tile_work_seconds(const pk_machine &m, const KernelEntry &e, int dtype, int64_t M, int64_t N, int64_t K,
                         int64_t res) {
    // compute-unit seconds of the product's tiles when the unit holds `res`
    // of this program's workgroups at a time: it advances them by one K step
    // in max(res * flops_step / rate, latency)
    const double clock = (m.clock_khz > 0 ? m.clock_khz : 2400000) * 1e3;
    const int wave = m.wave > 0 ? m.wave : 64;
    const int64_t tiles = ((M + e.tile_m - 1) / e.tile_m) * ((N + e.tile_n - 1) / e.tile_n);
    const int bk = e.bk > 0 ? e.bk : 1;
    const double ksteps = (double)((std::max<int64_t>(K, 1) + bk - 1) / bk);
    const double flops_step = 2.0 * e.tile_m * e.tile_n * bk;
    const double waves_per_simd = (double)res * ((e.threads + wave - 1) / wave) / 4.0;
    const double occupancy = std::min(1.0, std::pow(waves_per_simd / 3.0, 0.25));
    const bool mfma = e.family == PK_FAMILY_MFMA;
    const double eff = mfma ? 0.85 / (1.0 + 6.0 * (1.0 / e.tile_m + 1.0 / e.tile_n))
                            : std::min(1.0, e.threads / 256.0);
    const double rate = product_rate(m, e, dtype) * clock * eff * occupancy;
    const double latency = mfma ? ((e.variant & PK_MFMA_SINGLE) ? 0.4e-6 : 0.3e-6) : 0.1e-6;
    const double step = std::max((double)res * flops_step / rate, latency);
    return (double)tiles * ksteps * step / (double)res;
}

void fill_params(const pk_table *tbl, const Candidate &c, int dtype, pk_params *out) {
    const pk_table::Part *part = tbl->part(c.family, dtype);
    point_params(c.family, part->fam.points[c.point], out);
    out->leaf = c.leaf;
    out->variant = c.variant;
    out->ks = c.ks > 1 ? c.ks : 0;
}

std::vector<Candidate> feasible(const pk_table *tbl, int dtype, int64_t M, int64_t N, int64_t K, const void *A,
                                int64_t lda, const void *B, int64_t ldb) {
    std::vector<Candidate> out;
    out.reserve(192);
    for (int family : {PK_FAMILY_VALU, PK_FAMILY_VALU2, PK_FAMILY_MFMA}) {  // the product families
        const pk_table::Part *part = tbl->part(family, dtype);
        if (!part || !part->supported) continue;
        const int64_t ncu = std::max<int32_t>(tbl->machine.cu_count, 1);
        for (size_t i = 0; i < part->programs.size(); ++i) {
            const auto &p = part->programs[i];
            if (!p.entry) continue;
            // MFMA programs read unaligned rows at element alignment: feasible, slower
            const bool wide = !A || family != PK_FAMILY_MFMA || wide_rows(*p.entry, M, K, A, lda, B, ldb);
            if (!wide && !p.twin) continue;
            Candidate c;
            c.family = family;
            c.point = (int)i;
            c.leaf = part->first_leaf[i];
            c.variant = p.variant;
            c.entry = p.entry;
            c.estimate = estimate_program(tbl->machine, *p.entry, p.resident, p.rate, dtype, M, N, K, wide, 1);
            out.push_back(c);
            if (!p.split) continue;
            // the same program split along K: shares 2, 4, ... while the
            // product has fewer tiles than two per compute unit at the
            // previous count and every share keeps at least two K steps
            const KernelEntry &e = *p.entry;
            const int64_t tiles = ((M + e.tile_m - 1) / e.tile_m) * ((N + e.tile_n - 1) / e.tile_n);
            const int64_t ksteps = (K + e.bk - 1) / e.bk;
            for (int ks = 2; ks <= kMaxSplits && 2 * ks <= ksteps && tiles * (ks / 2) < 2 * ncu; ks *= 2) {
                Candidate d = c;
                d.ks = ks;
                d.estimate = estimate_program(tbl->machine, e, p.resident, p.rate, dtype, M, N, K, wide, ks);
                out.push_back(d);
            }
        }
    }
    return out;
}

// Times every candidate on the table's device.  Every HIP call is checked: a
// candidate whose launches or events fail is recorded as +inf (it can never
// be the pick), and a failure of the timing set-up itself is returned.
int time_candidates(const pk_table *tbl, int dtype, int64_t M, int64_t N, int64_t K,
                    const std::vector<Candidate> &cands, std::vector<double> *secs, const Operands *ops, int *best_out) {
    *best_out = -1;
    secs->assign(cands.size(), std::numeric_limits<double>::infinity());
    if (tbl->device < 0) return fail(PK_ERR_INVALID_ARG, "timing needs a table bound to a device");
    hipError_t err = hipSetDevice(tbl->device);
    if (err != hipSuccess) return fail(PK_ERR_HIP, std::string("hipSetDevice: ") + hipGetErrorString(err));
    const size_t es = dtype == PK_BF16 ? 2 : 4;
    void *sA = nullptr, *sB = nullptr, *sC = nullptr;
    hipStream_t s = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    auto release = [&]() {
        if (s) (void)hipStreamSynchronize(s);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
        if (s) (void)hipStreamDestroy(s);
        if (sA) (void)hipFree(sA);
        if (sB) (void)hipFree(sB);
        if (sC) (void)hipFree(sC);
    };
    auto setup_failed = [&](const char *what, hipError_t e) {
        release();
        return fail(PK_ERR_HIP, std::string("timing set-up, ") + what + ": " + hipGetErrorString(e));
    };
    MmArgs args{nullptr, nullptr, nullptr, K, N, N, (int32_t)M, (int32_t)N, (int32_t)K, 0, 0};
    if (ops && ops->A) {
        args.A = ops->A;
        args.B = ops->B;
        args.C = ops->C;
        args.lda = ops->lda;
        args.ldb = ops->ldb;
        args.ldc = ops->ldc;
    } else {
        // scratch operands with a non-zero byte pattern (0x3c: about 0.0115 in
        // float32 and bfloat16), so the timed kernels do real arithmetic
        const size_t bA = std::max<size_t>(es * M * K, 16), bB = std::max<size_t>(es * K * N, 16),
                     bC = std::max<size_t>(4 * M * N, 16);
        if ((err = hipMalloc(&sA, bA)) != hipSuccess) return setup_failed("hipMalloc", err);
        if ((err = hipMalloc(&sB, bB)) != hipSuccess) return setup_failed("hipMalloc", err);
        if ((err = hipMalloc(&sC, bC)) != hipSuccess) return setup_failed("hipMalloc", err);
        if ((err = hipMemset(sA, 0x3c, bA)) != hipSuccess) return setup_failed("hipMemset", err);
        if ((err = hipMemset(sB, 0x3c, bB)) != hipSuccess) return setup_failed("hipMemset", err);
        args.A = sA;
        args.B = sB;
        args.C = sC;
    }
    if ((err = hipStreamCreate(&s)) != hipSuccess) return setup_failed("hipStreamCreate", err);
    if ((err = hipEventCreate(&e0)) != hipSuccess) return setup_failed("hipEventCreate", err);
    if ((err = hipEventCreate(&e1)) != hipSuccess) return setup_failed("hipEventCreate", err);
    int best = -1;
    double best_t = std::numeric_limits<double>::infinity();
    // the most promising candidates first (least CASE estimate), so that the
    // best time so far is known early and slow candidates are cut short
    std::vector<size_t> order(cands.size());
    for (size_t i = 0; i < order.size(); ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(),
                     [&](size_t x, size_t y) { return cands[x].estimate < cands[y].estimate; });
    for (size_t i : order) {
        const KernelEntry &e = *cands[i].entry;
        MmArgs ca = args;
        ca.vec = wide_rows(e, M, K, args.A, args.lda, args.B, args.ldb) ? 1 : 0;
        ca.splits = cands[i].ks > 1 ? cands[i].ks : 0;
        // warm-up launch, itself timed: a candidate whose one launch already
        // takes over a millisecond (launch latency is then negligible) and
        // twice the best mean so far cannot win; its one-launch time is kept
        float wms = 0.f;
        if (hipEventRecord(e0, s) != hipSuccess || launch(tbl->machine, e, ca, s) != PK_OK ||
            hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&wms, e0, e1) != hipSuccess) {
            (void)hipGetLastError();
            (void)hipStreamSynchronize(s);
            continue;
        }
        if (wms > 1.f && wms * 1e-3 > 2.0 * best_t) {
            (*secs)[i] = wms * 1e-3;
            continue;
        }
        // back-to-back launches between two events, at least 3, up to about
        // 20 ms of work; after the first 3 a candidate already 1.5x slower
        // than the best so far cannot win and is not timed further (its mean
        // over those 3 is kept: a single launch between events would also
        // count the launch latency, which for small kernels exceeds the
        // kernel, and would cut off candidates that could win)
        float ms = 0.f;
        bool ok = hipEventRecord(e0, s) == hipSuccess;
        int reps = 0;
        while (ok) {
            ok = launch(tbl->machine, e, ca, s) == PK_OK;
            ++reps;
            if (ok && (reps == 3 || reps % 8 == 0)) {
                ok = hipEventRecord(e1, s) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
                     hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
                if (ok && reps == 3 && ms * 1e-3 / 3 > 1.5 * best_t) break;
            }
            if (reps >= 3 && (ms >= 20.f || reps >= 200)) break;
        }
        if (!ok || !(ms > 0.f)) {
            (void)hipGetLastError();  // this candidate only: leave it at +inf
            (void)hipStreamSynchronize(s);
            continue;
        }
        const double t = ms * 1e-3 / reps;
        (*secs)[i] = t;
        if (t < best_t) {
            best_t = t;
            best = (int)i;
        }
    }
    err = hipStreamSynchronize(s);
    release();
    if (err != hipSuccess) return fail(PK_ERR_HIP, std::string("timing: ") + hipGetErrorString(err));
    if (best < 0) return fail(PK_ERR_HIP, "no candidate could be launched and timed");
    *best_out = best;
    return PK_OK;
}

int select_params(const pk_table *tbl, int dtype, int64_t M, int64_t N, int64_t K, int policy, bool cache,
                  pk_params *out, const void *A, int64_t lda, const void *B, int64_t ldb) {
    const bool aligned_any = A == nullptr;
    auto key = std::make_tuple(dtype, M, N, K, policy);
    if (cache && aligned_any && tbl->cached(key, out)) return PK_OK;
    std::vector<Candidate> cands = feasible(tbl, dtype, M, N, K, A, lda, B, ldb);
    if (cands.empty()) return fail(PK_ERR_NO_FEASIBLE_BRANCH, "no leaf of the case table holds for this dtype");
    int pick = 0;
    const pk_costmodel *model = (dtype >= 0 && dtype < 3) ? tbl->costmodel[dtype].get() : nullptr;
    if (policy == PK_POLICY_LEARNED && model) {
        // order by predicted time; near-ties are settled by measurement
        std::vector<float> X(cands.size() * PK_NFEATURES), pred(cands.size());
        for (size_t i = 0; i < cands.size(); ++i)
            features(tbl->machine, *cands[i].entry, dtype, M, N, K,
                     !A || wide_rows(*cands[i].entry, M, K, A, lda, B, ldb), cands[i].ks, &X[i * PK_NFEATURES]);
        costmodel_predict(*model, tbl->device, X.data(), (int64_t)cands.size(), pred.data());
        std::vector<int> order(cands.size());
        for (size_t i = 0; i < order.size(); ++i) order[i] = (int)i;
        std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return pred[a] < pred[b]; });
        pick = order[0];
        tbl->learned_selections++;
        // candidates predicted within the table's margin of the best (5 % by
        // default) are too close for the model to order: they are measured
        const double margin = tbl->learned_margin;
        if (margin > 0.0 && order.size() > 1 && std::exp((double)pred[order[1]] - pred[order[0]]) < 1.0 + margin) {
            std::vector<Candidate> close;
            std::vector<int> idx;
            for (int i : order)
                if (std::exp((double)pred[i] - pred[order[0]]) <= 1.0 + margin) {
                    close.push_back(cands[i]);
                    idx.push_back(i);
                }
            std::vector<double> secs;
            Operands ops{A, lda, B, ldb, nullptr, 0};
            void *C = nullptr;
            if (A) {
                if (hipMalloc(&C, std::max<size_t>(4 * M * N, 16)) != hipSuccess)
                    return fail(PK_ERR_HIP, "learned selection: allocation failed");
                ops.C = C;
                ops.ldc = N;
            }
            int f = -1;
            const int rc = time_candidates(tbl, dtype, M, N, K, close, &secs, A ? &ops : nullptr, &f);
            if (C) (void)hipFree(C);
            if (rc != PK_OK) return rc;
            pick = idx[f];
            tbl->learned_fallbacks++;
            tbl->learned_measured += (int64_t)close.size();
        }
        fill_params(tbl, cands[pick], dtype, out);
    } else if (policy == PK_POLICY_CASE || policy == PK_POLICY_LEARNED) {
        for (size_t i = 1; i < cands.size(); ++i)
            if (cands[i].estimate < cands[pick].estimate) pick = (int)i;
        fill_params(tbl, cands[pick], dtype, out);
        if (policy == PK_POLICY_LEARNED)
            return fail(PK_ERR_COST_MODEL, "no cost model for this dtype loaded; CASE pick returned");
    } else if (policy == PK_POLICY_EXHAUSTIVE) {
        std::vector<double> secs;
        Operands ops{A, lda, B, ldb, nullptr, 0};
        void *C = nullptr;
        if (A) {  // time on the caller's data needs an output: scratch C
            if (hipMalloc(&C, std::max<size_t>(4 * M * N, 16)) != hipSuccess)
                return fail(PK_ERR_HIP, "exhaustive selection: allocation failed");
            ops.C = C;
            ops.ldc = N;
        }
        const int rc = time_candidates(tbl, dtype, M, N, K, cands, &secs, A ? &ops : nullptr, &pick);
        if (C) (void)hipFree(C);
        if (rc != PK_OK) return rc;
        fill_params(tbl, cands[pick], dtype, out);
    } else {
        return fail(PK_ERR_INVALID_ARG, "unknown policy");
    }
    if (cache && aligned_any) {
        std::lock_guard<std::mutex> g(tbl->cache_mu);
        tbl->cache[key] = *out;
    }
    return PK_OK;
}

}  // namespace pk
