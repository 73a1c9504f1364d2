// Which kernel a batched weight-streaming GEMM (1..64 rows) takes - host code only.
//
// Two kernels exist (dk_gemm.hip.h, dk_gemm_shared.hip.h).  Up to 16 batch rows the choice follows a few rules, given
// with both sides at gemm_plan_16().  Above, the choice between them, and the number of K slices of the second, comes
// from an estimate of each candidate's duration.  The estimate is a latency/occupancy model of a weight stream:
//
//   * a wave keeps a fixed number of bytes in flight, so a block streams at (waves x rate per wave)
//     until the compute units that are busy together reach the device's rate;
//   * the busiest compute unit works through ceil(blocks / compute units) blocks; blocks that are
//     resident together share its rate, blocks beyond that wait for a slot (one more block start);
//   * every 128-column step costs matrix-core and LDS time per 16-row batch tile that the stream does
//     not hide;
//   * a launch has a fixed cost, and K slices pay for the hand-over and the in-order sum of the
//     partial tiles.
//
// The constants were fitted (least squares on log time) to HBM-cold sweeps of both kernels over the
// layer matrices of the 0.6B, 3B, 8B and 30B-A3B shapes at 16..64 rows, 1..8 slices (about 400
// timings; the fit reproduces them to 13 % rms for the shared kernel, 16 % for the other).  What
// matters is the ranking: on those sweeps the estimate's choice is the measured best, or within 5 %
// of it, except where two candidates are within the sweeps' own scatter.  The sweeps are older than the 16-byte hand-over
// of K slices and the four-element stores of the epilogue, which shorten the fixed part of both kernels.
#pragma once
#include <algorithm>
#include <cmath>

namespace dkplan {

enum { EPI_STORE = 0, EPI_RESID = 1, EPI_SWIGLU = 2 };   // same values as dk::GEPI_*

struct GemmPlan { int w, slices; };   // w == 0: skinny_gemm_kernel; else shared_gemm_kernel, w waves per block

// Variant of skinny_gemm_kernel: MT 16-row batch tiles per block, KS waves that split K, RT row tiles per
// wave, `groups` groups of 16 batch rows across blockIdx.y (then MT == 1).
struct SkinnyVariant { int mt, ks, rt, groups; };

// Up to 16 batch rows what bounds a block is the bytes its compute unit fetches, about 40 GB/s of weights and
// activations together.
//   * Row tiles per wave: two - the activations once for both - where that leaves the busiest compute unit no more row
//     tiles than one each would: single matrices from more than one tile per compute unit on (3B shape, q/k/v, 320 tiles,
//     16 rows 15.3 -> 12.6 us; 288 tiles of K = 3072 and 3584 14.8 -> 12.4 and 17.2 -> 14.0, packed 13.6 -> 11.7; 0.6B shape,
//     256 tiles 5.2 -> 6.1), the gate/up pair between one and two (512 tiles 24.2 -> 21.9 us, 384 15.9 -> 14.3; 192 6.3 ->
//     8.4, 608 30.9 -> 35.1).
//   * Waves: four; a second block on the same compute unit hides the start and the end of the first, and steps that
//     do not divide among the waves cost less (eight -> four, 3B shape, K = 3072: gate/up 25.4 -> 21.9 us, q/k/v 14.1 ->
//     12.6; 4 rows with packed terms 23.7 -> 21.2 and 12.4 -> 11.0).  Unpacked terms: eight where a wave's two steps in
//     flight come out even (K = 2048: q/k/v 9.3 -> 8.9; 4 bit 7.3 -> 7.2, gate/up 10.3 -> 9.9; K = 4096, whole step of the 8B
//     shape, four / eight: 9 rows equal, 16 rows 1136 / 1133, 4 bit 707 / 703; K = 6144, 4 bit 556 / 544, bf16 825 / 831) or are
//     its only one (K = 1024, whole step of the 0.6B shape 1191 -> 1176), two for residual projections that make at most
//     one block per compute unit (less to add up: K = 2048 6.4 -> 6.3, 4096 11.0 -> 10.8).
// Above 16 rows: a small matrix whose row tiles x groups of 16 rows still make at most two blocks per compute unit runs
// the 16-row kernel over all groups at once, residual projections with two-wave blocks; with 4-bit weights
// and more than 48 rows, residual projections of up to three blocks as well, of four waves (a wave's steps and the order of
// their sums are those of the 64-row block; 64 rows, 192 row tiles of K = 3072 14.8 -> 12.6 us; whole steps of 12 layers
// with 136, 144, 160, 192 tiles 846 -> 803, 1249 -> 1170, 1449 -> 1409, 1036 -> 978).  Not up to 48 rows, whose own block
// leaves less to gain (whole steps: 192 tiles, 48 rows 894 / 908 and 2434 / 2437, 40 rows 1201 / 1195; 224 tiles 1730 /
// 1743; 256 tiles, 48 rows 1140 / 1169, 8B shape 4238 / 4265, 33 rows 1115 / 1141).
inline SkinnyVariant skinny_variant(int epi, int N, int K, int Bp, bool q4, bool pack, int cus)
{
    const int tiles = (N + 15) / 16, mt = Bp / 16;
    const bool one_matrix = epi != EPI_SWIGLU;
    if (mt == 1) {
        const bool two = tiles > cus && (one_matrix || tiles <= 2 * cus);
        if (!pack && epi == EPI_RESID && !q4 && tiles <= cus) return {1, 2, 1, 1};
        return {1, !pack && (K <= 1024 || K % 2048 == 0) ? 8 : 4, two ? 2 : 1, 1};
    }
    if (tiles * mt <= 2 * cus) return {1, epi == EPI_RESID && !q4 ? 2 : 8, 1, mt};
    if (mt == 4 && q4 && epi == EPI_RESID && tiles * mt <= 3 * cus) return {1, 4, 1, mt};
    switch (mt) {
        case 2:
            if (one_matrix && tiles >= 4 * cus) return {2, 8, 2, 1};
            return {2, 8, 1, 1};
        case 3: return {3, 4, 1, 1};
        default: return {4, 4, 1, 1};
    }
}

// ---- estimates, in microseconds (bf16 weights) ---------------------------------------------------
constexpr double kStepBytes = 4096.0;        // one 16-row x 128-column weight tile
// shared_gemm_kernel
constexpr double kShLaunch = 5.78;           // launch, first loads, epilogue
constexpr double kShBlockStart = 0.58;       // per block that starts on a busy compute unit
constexpr double kShWaveRate = 16.4e3;       // bytes per us a wave streams (two steps in flight)
constexpr double kShDeviceRate = 7.04e6;     // bytes per us all compute units together
constexpr double kShTileStep = 0.22;         // us per step, 16-row batch tile and matrix (not hidden)
constexpr double kShSliceTile = 0.18;        // us per slice, batch tile and matrix for the hand-over
// skinny_gemm_kernel
constexpr double kSkLaunch = 2.06;
constexpr double kSkWaveRate = 89.1e3;       // a lone wave is not the limit: the compute unit is
constexpr double kSkCuRate = 37.6e3;         // bytes per us the waves of one compute unit stream together
constexpr double kSkDeviceRate = 6.41e6;
constexpr double kSkActShare = 0.47;         // a wave's own activation fetch (8 KB per batch tile and step), as stream bytes
constexpr double kSkTileStep = 0.036;
constexpr double kSkReduce = 0.176;          // us per wave, batch tile, row tile and matrix summed through LDS
constexpr double kSkWavesPerCu = 32.0;       // resident waves per compute unit

inline double shared_gemm_us(int N, int K, int n_mat, int mt, int w, int slices, int cus)
{
    const int tiles = (N + 15) / 16, row_blocks = (tiles + w - 1) / w, blocks = row_blocks * slices;
    const int steps = (K / 128 + slices - 1) / slices;
    const int occ = w <= 4 ? 2 : 1;                             // blocks resident per compute unit
    const int active = std::min(cus, blocks);
    const int per_cu = (blocks + cus - 1) / cus;                // blocks of the busiest compute unit
    const int resident = std::min(occ, per_cu);
    const double rate = std::min(kShWaveRate * w * resident, kShDeviceRate / active);
    double t = kShLaunch + kShBlockStart * ((per_cu + occ - 1) / occ) +
               (double)steps * per_cu * (w * n_mat * kStepBytes / rate + kShTileStep * mt * n_mat / resident);
    if (slices > 1) t += kShSliceTile * slices * mt * n_mat;
    return t;
}

inline double skinny_gemm_us(int N, int K, int n_mat, const SkinnyVariant &v, int cus)
{
    const int tiles = (N + 15) / 16;
    const double blocks = (double)((tiles + v.rt - 1) / v.rt) * v.groups;
    const double slots = cus * std::max(1.0, kSkWavesPerCu / v.ks);
    const double rounds = std::max(1.0, blocks / slots);
    const int steps = ((K + 127) / 128 + v.ks - 1) / v.ks;
    const double conc = std::min(blocks, slots), active = std::min((double)cus, conc), per_cu = conc / active;
    const double wave_step = v.rt * n_mat * kStepBytes + kSkActShare * v.mt * 2.0 * kStepBytes;
    const double rate = std::min(std::min(kSkWaveRate, kSkCuRate / (per_cu * v.ks)), kSkDeviceRate / (active * per_cu * v.ks));
    return kSkLaunch + rounds * steps * (wave_step / rate + kSkTileStep * v.mt * v.rt * n_mat) +
           kSkReduce * v.ks * v.mt * v.rt * n_mat;
}

// K slices of shared_gemm_kernel for blocks of w waves: as many as still give one round of blocks on the
// compute units (a second, partly filled round costs more than the slices save), at least four K-steps per
// slice, at most 8; a matrix whose row blocks alone fill more than half the chip takes four.
inline int shared_gemm_slices(int N, int K, int w, int cus)
{
    const int row_blocks = ((N + 15) / 16 + w - 1) / w;
    if (row_blocks > cus / 2) return std::max(1, std::min(4, K / 512));
    return std::max(1, std::min(std::min(cus / row_blocks, 8), K / 512));
}

// 4-bit weights above 16 rows: thresholds from a sweep of the 4-bit kernels over the same shapes (their streams are a
// quarter as long and their steps carry the dequantisation, which this model's constants do not cover):
// the lm_head at every batch size; q | k | v from 32 rows on; the gate/up pair and the down projection of
// the 3B / 8B shapes; never the output projection.
inline GemmPlan gemm_plan_q4(int epi, int N, int K)
{
    const long long elems = (long long)N * K;
    if (epi == EPI_STORE) {
        if ((N + 15) / 16 >= 4096) return {8, 1};
        if (elems >= (8ll << 20)) return {8, 4};
    } else if (epi == EPI_SWIGLU) {
        if (elems >= (40ll << 20)) return {8, 2};
        if (elems >= (20ll << 20)) return {8, 4};
    } else {
        if (elems >= (20ll << 20)) return {4, 8};
    }
    return {0, 1};
}

// Up to 16 batch rows.  Sweep of the 3B, 8B, 0.6B, 30B-A3B layer matrices and of layers of 2560 x 9728 and 1536 x 8960;
// `pack`: the terms of an activation share one operand, so the activations, which a wave of skinny_gemm_kernel fetches
// for itself, are half as many bytes and the line moves.  us, skinny / shared:
//   * long residual projections, whose few row tiles leave a compute unit one long block, are cut into K slices:
//     K = 6144 14.4 / 11.2, 8192 18.2 / 14.0, 12288 27.7 / 22.3, K = 4096 equal, 3072 8.8 / 9.0; packed 8192 14.2 / 13.9,
//     12288 equal, 6144 equal, 4096 8.8 / 10.8; 4 bit 8192 13.2 / 12.5, 12288 19.0 / 16.1, 6144 equal; 4 bit packed
//     never (8192 9.4 / 12+);
//   * gate/up pairs of more than two row tiles per compute unit: 608 tiles 30.9 / 25.3, 768 equal; packed only where the
//     tiles do not fill their rounds of blocks (608: 26.7 / 24.7, 768: 37.0 / 42.0); 4 bit 608 17.6 / 15.3, 768 24.4 / 21.9,
//     packed 768 equal.  Slices: the count that fills the compute units best (608 tiles, 3 / 4 / 5 slices: 25.3 / 29.3 /
//     25.3 us; 768 tiles, 2 / 3 / 4 / 5: 46.7 / 48.9 / 42.2 / 46.0), the smaller one where that fills them within 15 % as
//     well (576 tiles of K = 3072, 3 / 5: 26.6 / 29.9; 592 30.7 / 31.6; 1376 of K = 8192, 2 / 5: 139.6 / 141.3; 4 bit, 1184
//     tiles, 3 / 5, whole step of layers of 3584 x 18944 275 / 291); one where a stream is short (K = 2048, 688 tiles, 1 / 4:
//     21.5 / 24.9, 864 tiles, 1 / 2: 22.7 / 28.3, packed 22.2 / 28.0; K = 1536, 560 tiles, 1 / 3: equal; K = 2304, 576 tiles
//     24.4 / 21.5);
//   * the lm_head, where the stream is long enough for one slice: 151936 x 1024 60 / 53, x 4096 237 / 212; packed 50 / 53,
//     205 / 211; 4 bit 36 / 30, 132 / 100, packed 30 / 25, 101 / 87;
//   * shorter plain stores of three and four row tiles per compute unit, which two tiles per wave fill badly, in slices:
//     640 tiles of K = 8192 52.1 / 34.4, 1000 of K = 2560 23.6 / 20.8, 3584 29.2 / 25.3, 5120 39.5 / 35.6, 8192 62.0 / 50.0 (K =
//     2048 and 4096 16.8 / 17.4 and 29.3 / 31.0); 512 tiles of K = 6144 equal, 448 of K = 5120 20.6 / 20.0.
inline GemmPlan gemm_plan_16(int epi, int N, int K, bool q4, bool pack, int cus)
{
    const int tiles = (N + 15) / 16;
    if (epi == EPI_STORE) {
        if (q4) return tiles >= 16 * cus ? GemmPlan{8, 1} : GemmPlan{0, 1};
        if (pack || tiles <= 2 * cus) return {0, 1};
        return {8, tiles >= 4 * cus ? 1 : shared_gemm_slices(N, K, 8, cus)};
    }
    if (epi == EPI_RESID) {
        if (K < (q4 || pack ? 8192 : 4097) || (q4 && pack)) return {0, 1};
        return {4, q4 ? 8 : shared_gemm_slices(N, K, 4, cus)};
    }
    const int rounds = (tiles + cus - 1) / cus;
    if (rounds <= 2 || (pack && (q4 || tiles * 20 >= rounds * cus * 17))) return {0, 1};
    const int w = q4 ? 8 : 4, row_blocks = (tiles + w - 1) / w;
    GemmPlan best{w, 1};
    if (row_blocks >= 2 * cus || (!q4 && K <= 2048)) return best;
    double best_fill = 0.0;
    for (int s = 2; s <= std::min(5, K / 512); s++) {
        const int blocks = row_blocks * s;
        const double fill = (double)blocks / ((double)cus * ((blocks + cus - 1) / cus));
        if (fill > 1.15 * best_fill) { best_fill = fill; best.slices = s; }
    }
    return best;
}

// Waves per block a plan runs with.  Gate/up pairs of more than 16 rows that are planned with eight take six where the
// busiest compute unit then gets fewer row tiles: the 8B shape's 768 tiles in two slices are 192 blocks of eight, three
// quarters of the chip, or 256 of six (64 rows 61.0 -> 54.8 us; 688 tiles 58.0 -> 52.2; 1088 tiles in four slices, three
// rounds of blocks either way, whole step of layers of 5120 x 17408 1639 -> 1581; the 3B shape's 512 tiles in four
// slices fill the chip with eight: 30.8, with six 40.4).  Sums and their order are the same.
inline int shared_waves(int epi, int N, int mt, const GemmPlan &p, int cus)
{
    if (epi != EPI_SWIGLU || mt < 2 || p.w != 8) return p.w;
    const int tiles = (N + 15) / 16;
    auto busiest = [&](int w) { return ((tiles + w - 1) / w * p.slices + cus - 1) / cus * w; };
    return busiest(6) < busiest(8) ? 6 : 8;
}

// The plan.  Above 16 rows: the candidate with the smallest estimate.  Candidates are the skinny kernel (its variant by
// skinny_variant) and the shared kernel in the block widths that are instantiated for the epilogue - 8
// waves for plain stores and the gate/up pair, 4 waves for residual projections -
// with shared_gemm_slices() slices (one slice when the row blocks alone make several rounds: the lm_head).
// est_us (optional) receives the estimate for the plan.
inline GemmPlan gemm_plan(int epi, int N, int K, int Bp, bool q4, bool pack, int cus, double *est_us = nullptr)
{
    const int mt = Bp / 16;
    if (est_us) *est_us = 0.0;
    if (K % 128) return {0, 1};
    const int n_mat = epi == EPI_SWIGLU ? 2 : 1;
    if (mt == 1) {
        const GemmPlan p = gemm_plan_16(epi, N, K, q4, pack, cus);
        if (est_us && !q4)
            *est_us = p.w ? shared_gemm_us(N, K, n_mat, 1, p.w, p.slices, cus)
                          : skinny_gemm_us(N, K, n_mat, skinny_variant(epi, N, K, Bp, false, pack, cus), cus);
        return p;
    }
    if (q4) return gemm_plan_q4(epi, N, K);
    GemmPlan best{0, 1};
    double best_us = skinny_gemm_us(N, K, n_mat, skinny_variant(epi, N, K, Bp, false, pack, cus), cus);
    const int w = epi == EPI_RESID ? 4 : 8, row_blocks = ((N + 15) / 16 + w - 1) / w;
    const int s = row_blocks >= 2 * cus ? 1 : shared_gemm_slices(N, K, w, cus);
    const double us = shared_gemm_us(N, K, n_mat, mt, w, s, cus);
    if (us < best_us) { best_us = us; best = {w, s}; }
    if (est_us) *est_us = best_us;
    return best;
}

}  // namespace dkplan
