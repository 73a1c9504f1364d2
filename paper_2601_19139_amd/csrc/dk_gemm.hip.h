// Weight-streaming skinny GEMM on the matrix cores: 5..64 rows, three and four of the larger dense models, and every
// count of expert and 4-bit models.
//
//   D[r][n] = sum_k W[r][k] * X[n][k]          r: weight row, n: batch row
//
// One 16x16x32 bf16 MFMA takes a 16-row x 32-k weight tile as its A operand
// and 32 k x 16 batch rows as its B operand, so the weights go from the global
// load straight into the MFMA with no vector-ALU work at all, and each weight
// byte is still read from HBM exactly once.  The activations stay accurate:
// they are kept as two bf16 numbers hi + lo (hi = bf16(x), lo = bf16(x - hi),
// about 16 significant bits; three or four rows as three numbers, all 24 bits)
// and each weight tile is multiplied by every one - the
// matrix cores have an order of magnitude more throughput than the HBM stream
// needs, so the second product is free; up to eight rows one product does for all (kPackCols).
//
// A block owns a group of 16*RT weight rows (SWIGLU: of each of the two
// matrices); its KS waves split K in interleaved 128-element steps (a lane loads 64
// contiguous bytes of one row per step, the wave 16 rows x 256 bytes) and add
// their accumulators through LDS in a fixed order.  The activations are stored
// in the order the B-operand loads consume them (act_offset), so each of those
// loads is one contiguous 1 KB run per wave.  With NORM the RMSNorm of
// the input is fused: the producer stored (x * gain) as hi/lo plus per-tile
// sums of x^2; the scalar 1/rms per batch row is applied in the epilogue.
//
// Q4: the weights are 4-bit codes with a bf16 scale and bias per group of 64
// columns (w = scale * q + bias).  A lane's 16-byte load then carries a whole
// K-step (32 codes) of its row.  The product is evaluated exactly as
//   sum_g ( scale_g * sum_{k in g} q_k x_k  +  bias_g * sum_{k in g} x_k ):
// the codes go to the matrix cores as the bf16 numbers 0..15, a second product
// with an all-ones operand gives the group sums of x, and fused multiply-adds
// apply scale and bias to the fp32 tiles.  (Feeding the codes as 128 + q, which
// is a two-instruction bit pattern, was measured to cost three decimal digits:
// the matrix cores do not keep the full fp32 sum while adding products, and the
// offset term, 17 times the useful one, has to cancel afterwards.)
#pragma once
#include "dk_common.hip.h"

namespace dk {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

enum { GEPI_STORE = 0, GEPI_RESID = 1, GEPI_SWIGLU = 2 };

constexpr int kSsqStride = 64;  // floats per row of the sum-of-squares partial table

struct GemmArgs {
    const uint16_t *W;       // [N][K] bf16; Q4: the packed 4-bit matrix (codes, then scale/bias tiles)
    const uint16_t *W2;      // GEPI_SWIGLU: the "up" matrix, same format as W
    int N, K, B;             // B valid batch rows (<= 16*MT)
    int q4;                  // host side only: W / W2 are packed 4-bit matrices (selects the Q4 kernels)
    int spread;              // shared_gemm_kernel, more than 16 rows: blocks may begin at columns of their own
    int pack;                // host side only: the terms of an activation share one operand (2 or 3, see kPackCols)
    const uint16_t *xhi;     // hi part of the input, bf16 in act_offset() order
    const uint16_t *xlo;     // lo part
    // NORM: sum over p < n_part of ssq_in[p][n] = sum_k x[n][k]^2
    const float *ssq_in;
    int n_part;
    float eps;
    // GEPI_STORE: y[B][N] (may be null), optional running maxima [B][ceil(N/16)]
    float *y;
    float *pmax_val;
    int *pmax_idx;
    // GEPI_SWIGLU and GEPI_RESID: result as hi/lo bf16 in act_offset() order (K = N)
    // for the next GEMM
    uint16_t *ohi, *olo;
    uint16_t *ox3;           // three terms: the third one
    // GEPI_RESID: xres[B][N] += D; the hi/lo output is (xres * gain_next); the
    // sum of xres^2 over each 16-row tile and batch row goes to ssq_out[tile][n]
    float *xres;
    const uint16_t *gain_next;  // [N]
    float *ssq_out;
    // shared_gemm_kernel with K cut into slices: partial tiles and one ticket per row block
    // (zero before the launch, zero after)
    float *kpart;
    int *ktickets;
    // shared_gemm_kernel, q | k | v of a prompt chunk whose blocks hold a head each (heads of 128, eight waves): q_heads > 0,
    // and the k and v heads go to the pool instead of y
    int q_heads, kv_heads;
    const float2 *cs;        // [B][64]
    const uint16_t *g_k;     // [128] or null
    uint16_t *pool;
    const int *block_table, *seq_lens;
    int max_blocks, num_blocks, layer;
};

__device__ __forceinline__ void split_bf16(float x, uint16_t &hi, uint16_t &lo)
{
    hi = f32_to_bf16_rne(x);
    lo = f32_to_bf16_rne(x - bf16_to_f32(hi));
}

// the same for two values: a in the low half-words of hi / lo, b in the high ones
__device__ __forceinline__ void split_bf16x2(float a, float b, uint32_t &hi, uint32_t &lo)
{
    hi = f32x2_to_bf16x2_rne(a, b);
    lo = f32x2_to_bf16x2_rne(a - bf16lo(hi), b - bf16hi(hi));
}

// x = hi + mid + lo: all 24 bits of a float32
__device__ __forceinline__ void split_bf16x3(float x, uint16_t &hi, uint16_t &mid, uint16_t &lo)
{
    hi = f32_to_bf16_rne(x);
    const float r = x - bf16_to_f32(hi);
    mid = f32_to_bf16_rne(r);
    lo = f32_to_bf16_rne(r - bf16_to_f32(mid));
}

// Few batch rows: a 16-column operand holds all terms of every row side by side - term i of row n in column
// i * kPackCols(terms) + n, so up to eight rows of two terms or five of three.  One matrix product then does what two
// (three) did, the activations are half (a half) of the bytes, and a row's terms are added up across the columns
// afterwards.  In act_offset() order the next term of a row lies kPackCols * 8 elements further on: writers only see
// other pointers.  Columns that belong to no row hold whatever the buffer held; a column never meets another.
constexpr int kPackCols(int terms) { return terms == 2 ? 8 : 5; }

// The sum over a row's terms, smallest first, for the lane of the row's first column.
template <int PACK>
__device__ __forceinline__ float pack_sum(float v, int lane)
{
    if (PACK == 0) return v;
    const int row = lane & 48, ln = lane & 15;
    const float v1 = __shfl(v, row | ((ln + kPackCols(PACK)) & 15));
    if (PACK == 2) return v1 + v;
    const float v2 = __shfl(v, row | ((ln + 2 * kPackCols(PACK)) & 15));
    return (v2 + v1) + v;
}

__device__ __forceinline__ bf16x8_t as_bf16x8(const uint4 &u)
{
    union { uint4 u; bf16x8_t v; } c;
    c.u = u;
    return c.v;
}

// The eight 4-bit codes of a word (code j in bits 4j..4j+3) as exact bf16 numbers, in matrix-core operand
// order.  A byte 0..15 read as an fp8 (e4m3) number is exactly code * 2^-9: the codes below 8 are its subnormals,
// the others its first binade.  So the gfx950 conversion of two fp8 numbers to bf16 with a scale of 2^9 yields two
// codes per instruction: nibbles to bytes in column order (5 instructions) and four conversions, against 15
// instructions by way of float (checked on the device for every pair of codes: identical bits).  4-bit 3B shape:
// 2.136 -> 2.092 ms per step at 16 rows, 700-token prefill 38.5 -> 37.5 ms.
__device__ __forceinline__ uint4 q4_codes_bf16(uint32_t w)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    const uint32_t ev = w & 0x0F0F0F0Fu, od = (w >> 4) & 0x0F0F0F0Fu;
    const uint32_t lo = __builtin_amdgcn_perm(od, ev, 0x05010400u);   // columns 0, 1, 2, 3
    const uint32_t hi = __builtin_amdgcn_perm(od, ev, 0x07030602u);   // columns 4, 5, 6, 7
    const bf16x2_t c[4] = {__builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.f, false),
                           __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.f, true),
                           __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.f, false),
                           __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.f, true)};
    uint4 r;
    __builtin_memcpy(&r, c, 16);
    return r;
}

// The four residual values xres[n][r .. r+3] of a lane.  r and N are multiples of 4; rows past the end are clamped:
// valid addresses, unused values.
__device__ __forceinline__ void load_resid4(const float *xrow, int r, int N, float (&x)[4])
{
    const float4 v = ldf4(xrow + min(r, N - 4));
    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
}

// Epilogue of one finished 16-row tile.  The lane holds D[row0 + 4*lg + i][n = 16*t + ln], i = 0..3, in
// v[t][matrix][i] (already scaled by 1/rms where the input norm is fused).  xr / gn: the residual rows and the
// next norm's gains of exactly those elements (GEPI_RESID; loaded by the caller ahead of the weight stream).
// A lane's four rows lie side by side in every output (act_offset keeps runs of 8 columns together) and leave in one
// store each: 8 bytes for the hi and the lo half, 16 for float32, a quarter of the requests on the tail of the
// kernel (501-token prefill of the 8B shape 48.7 -> 45.7 ms, 700 tokens of the 3B shape with 4-bit weights 37.5 ->
// 34.9, 16 rows of it 2.12 -> 2.08 ms per step).  For GEPI_RESID and GEPI_SWIGLU N is the model's hidden or ffn size,
// a multiple of 8 (checked where a model is created, and at the launch).  Only logits (GEPI_STORE) can have another
// N or an address that is not 16-byte aligned; those go element by element.  A narrow path in the other two, which
// nothing reached, cost registers and branches there: 16 rows of the 0.6B shape 1225 -> 1200 us per step without it,
// 700 tokens of the 3B shape with 4-bit weights 34.4 -> 33.5 ms.
template <int MT, int EPI, int PACK = 0>
__device__ __forceinline__ void gemm_tile_epilogue(const GemmArgs &a, int out_tile, int lane,
                                                   const float (&v)[MT][(EPI == GEPI_SWIGLU) ? 2 : 1][4],
                                                   const float (&xr)[MT][4], const float (&gn)[4])
{
    constexpr int NM = (EPI == GEPI_SWIGLU) ? 2 : 1;
    const int ln = lane & 15, lg = lane >> 4;
    const int N = a.N;
    const int onks = (N + 127) >> 7;   // K-steps of the GEMM that consumes this output
    const int n_tiles = (N + 15) >> 4;
    const int row0 = out_tile * 16;
    const bool wide = EPI != GEPI_STORE || ((N & 3) == 0 && ((uintptr_t)a.y & 15) == 0);
    float best = -INFINITY;
    int best_i = 0x7fffffff;
#pragma unroll
    for (int t = 0; t < MT; t++) {
        const int n = t * 16 + ln;
        const bool nvalid = n < a.B;
        const int rr = row0 + 4 * lg;
        float sq = 0.f;
        float out[4];
        uint32_t hi[2], lo[2], x3[2];   // two elements a word
#pragma unroll
        for (int i = 0; i < 4; i++) {
            if (EPI == GEPI_SWIGLU) {
                const float z = v[t][0][i];
                out[i] = z / (1.0f + __expf(-z)) * v[t][NM - 1][i];
            } else {
                out[i] = EPI == GEPI_RESID ? xr[t][i] + v[t][0][i] : v[t][0][i];
            }
        }
        if (EPI != GEPI_STORE) {
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const float g0 = EPI == GEPI_RESID ? gn[2 * h] : 1.f, g1 = EPI == GEPI_RESID ? gn[2 * h + 1] : 1.f;
                if constexpr (PACK == 3) {
                    uint16_t t[2][3];
                    split_bf16x3(out[2 * h] * g0, t[0][0], t[0][1], t[0][2]);
                    split_bf16x3(out[2 * h + 1] * g1, t[1][0], t[1][1], t[1][2]);
                    hi[h] = t[0][0] | (uint32_t)t[1][0] << 16;
                    lo[h] = t[0][1] | (uint32_t)t[1][1] << 16;
                    x3[h] = t[0][2] | (uint32_t)t[1][2] << 16;
                } else {
                    split_bf16x2(out[2 * h] * g0, out[2 * h + 1] * g1, hi[h], lo[h]);
                }
            }
        }
        if (wide && nvalid && rr < N) {
            if (EPI == GEPI_STORE) {
                if (a.y != nullptr)
                    *reinterpret_cast<float4 *>(a.y + (int64_t)n * N + rr) = make_float4(out[0], out[1], out[2], out[3]);
            } else {
                const int64_t oo = act_offset(n, rr, onks);
                *reinterpret_cast<uint2 *>(a.ohi + oo) = make_uint2(hi[0], hi[1]);
                *reinterpret_cast<uint2 *>(a.olo + oo) = make_uint2(lo[0], lo[1]);
                if (PACK == 3) *reinterpret_cast<uint2 *>(a.ox3 + oo) = make_uint2(x3[0], x3[1]);
                if (EPI == GEPI_RESID)
                    *reinterpret_cast<float4 *>(a.xres + (int64_t)n * N + rr) = make_float4(out[0], out[1], out[2], out[3]);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int r = rr + i;
            if (!nvalid || r >= N) continue;
            if (EPI == GEPI_STORE && out[i] > best) { best = out[i]; best_i = r; }
            if (EPI == GEPI_RESID) sq += out[i] * out[i];
            if (!wide && a.y != nullptr) a.y[(int64_t)n * N + r] = out[i];
        }
        if (EPI == GEPI_RESID) {
            // the tile's 16 rows of batch row n are spread over the 4 lane groups
            sq += __shfl_xor(sq, 16);
            sq += __shfl_xor(sq, 32);
            if (lg == 0) a.ssq_out[(int64_t)out_tile * kSsqStride + n] = nvalid ? sq : 0.f;
        }
        if (EPI == GEPI_STORE && a.pmax_val != nullptr) {
#pragma unroll
            for (int off = 16; off < 64; off <<= 1) {
                const float ov = __shfl_xor(best, off);
                const int oi = __shfl_xor(best_i, off);
                if (ov > best || (ov == best && oi < best_i)) { best = ov; best_i = oi; }
            }
            if (lg == 0 && nvalid) {
                a.pmax_val[(int64_t)n * n_tiles + out_tile] = best;
                a.pmax_idx[(int64_t)n * n_tiles + out_tile] = best_i;
            }
            best = -INFINITY;
            best_i = 0x7fffffff;
        }
    }
}

// The sum-of-squares partials of the input rows (NORM), for one of NW waves that share them; a partial is a row of
// kSsqStride floats.  request() comes ahead of the first weights, store() - out[0..16*MT) - behind their requests, so
// that the sums are made while the weights are under way.  Up to 16 batch rows a load brings 16 partials (16 bytes a
// lane, four lanes to a partial): one float a lane and load was 16 times as many requests, all of them in front of
// the first weights, and loads return in order (shared_gemm_kernel, 16 rows, blocks of four waves, gate/up of 9472 x 3584
// 33.2 -> 29.9 us, 8960 x 1536 16.8 -> 16.3; blocks of eight the same).  Beyond 16 rows the same measured nothing.
template <int MT, int NW>
struct SsqPartials {
    static constexpr int U = MT == 1 ? 4 : 32;   // loads held in registers
    float4 q[MT == 1 ? U : 1];
    float v[MT == 1 ? 1 : U];
    __device__ __forceinline__ int part(int wv, int lane, int u) const
    {
        return MT == 1 ? (u * NW + wv) * 16 + (lane >> 2) : u * NW + wv;
    }
    __device__ __forceinline__ void request(const float *ssq, int n_part, int wv, int lane)
    {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const float *row = ssq + (int64_t)min(part(wv, lane, u), n_part - 1) * kSsqStride;
            if constexpr (MT == 1) q[u] = ldf4(row + (lane & 3) * 4);
            else v[u] = row[min(lane, 16 * MT - 1)];
        }
    }
    __device__ __forceinline__ void store(const float *ssq, int n_part, int wv, int lane, float *out)
    {
        if constexpr (MT == 1) {
            float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
            auto add = [&](const float4 &w) { s.x += w.x; s.y += w.y; s.z += w.z; s.w += w.w; };
#pragma unroll
            for (int u = 0; u < U; u++)
                if (part(wv, lane, u) < n_part) add(q[u]);
            for (int p = part(wv, lane, U); p < n_part; p += NW * 16)   // very wide models only
                add(ldf4(ssq + (int64_t)p * kSsqStride + (lane & 3) * 4));
#pragma unroll
            for (int off = 4; off < 64; off <<= 1) {
                s.x += __shfl_xor(s.x, off);
                s.y += __shfl_xor(s.y, off);
                s.z += __shfl_xor(s.z, off);
                s.w += __shfl_xor(s.w, off);
            }
            if (lane < 4) *reinterpret_cast<float4 *>(out + lane * 4) = s;
        } else {
            float s = 0.f;
#pragma unroll
            for (int u = 0; u < U; u++) s += part(wv, lane, u) < n_part ? v[u] : 0.f;
            for (int p = part(wv, lane, U); p < n_part; p += NW) s += ssq[(int64_t)p * kSsqStride + min(lane, 16 * MT - 1)];
            out[lane] = s;
        }
    }
};

// KALIGNED: K is a multiple of 128 (every real model shape); the K-steps are then
// whole and the loaded registers feed the MFMAs untouched.
// Q4 (needs KALIGNED): per row K/2 bytes of codes, a K-step of 128 columns being 16 words
// [lane group lg][sub-step s] whose nibble j (bits 4j..4j+3) is column s*32 + lg*8 + j;
// after the N rows, per 16-row tile and K-step 128 bytes [lg][group h of the step][row 4*lg+i]
// of (scale, bias) bf16 pairs - the order in which the accumulator lanes need them.
// PACK (MT = 1, KALIGNED): xhi is one operand with PACK terms of every row (kPackCols).
template <int MT, int KS, int RT, int PD, int EPI, bool NORM, bool KALIGNED, bool Q4 = false, int PACK = 0>
__global__ __launch_bounds__(KS * 64) void skinny_gemm_kernel(GemmArgs a)
{
    static_assert(PACK == 0 || (MT == 1 && KALIGNED && !(Q4 && PACK == 3)), "packed terms fill one 16-column operand");
    static_assert(!Q4 || KALIGNED, "4-bit weights need whole K-steps");
    constexpr int NM = (EPI == GEPI_SWIGLU) ? 2 : 1;
    constexpr int NA = NM * RT;   // weight tiles (accumulator sets) per wave
    static_assert(KS * NA * MT <= 32, "LDS reduction buffer is limited to 32 KB");
    extern __shared__ float dyn_lds[];
    typedef float RedBuf[KS][NA][MT][4][64];
    RedBuf *red = reinterpret_cast<RedBuf *>(dyn_lds);
    float (*ssq_s)[64] = reinterpret_cast<float (*)[64]>(dyn_lds + sizeof(RedBuf) / sizeof(float));

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index, known to be uniform
    const int ln = lane & 15, lg = lane >> 4;
    const int K = a.K, N = a.N;
    const int nks = (K + 127) >> 7;
    if (gridDim.y > 1) {
        // The batch rows are split across blockIdx.y in groups of 16*MT: a small matrix (few row
        // tiles) then still gives every compute unit a block, each with a quarter of the epilogue,
        // and the weights, read once per group, stay in the caches.  Every table is tile-major or
        // row-major in the batch row, so a group is the same problem behind shifted pointers.
        const int ct = (int)blockIdx.y * MT;   // first column tile of this block
        const int64_t onks = (N + 127) >> 7, n_tiles = (N + 15) >> 4;
        a.xhi += (int64_t)ct * nks * 2048;
        a.xlo += (int64_t)ct * nks * 2048;
        if (NORM) a.ssq_in += 16 * ct;
        if (EPI == GEPI_STORE) {
            if (a.y != nullptr) a.y += (int64_t)16 * ct * N;
            if (a.pmax_val != nullptr) {
                a.pmax_val += (int64_t)16 * ct * n_tiles;
                a.pmax_idx += (int64_t)16 * ct * n_tiles;
            }
        } else {
            a.ohi += (int64_t)ct * onks * 2048;
            a.olo += (int64_t)ct * onks * 2048;
        }
        if (EPI == GEPI_RESID) {
            a.xres += (int64_t)16 * ct * N;
            a.ssq_out += 16 * ct;
        }
        a.B = min(16 * MT, a.B - 16 * ct);
    }
    const int niter = (nks + KS - 1) / KS;   // K-steps per wave and row group
    const int niter2 = (niter + PD - 1) / PD * PD;   // padded to the pipeline depth

    f32x4_t acc[NA][MT];
#pragma unroll
    for (int m = 0; m < NA; m++)
#pragma unroll
        for (int t = 0; t < MT; t++) acc[m][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Software pipeline: PD K-steps are always in flight per wave.  The loop has
    // no conditional loads and no stores (the compiler can then wait for exactly
    // the stage it is about to use): every wave runs the same number of steps, a
    // multiple of PD; a step past the end of K reads clamped (valid, cached)
    // addresses and is not used.
    struct Stage {
        uint4 wa[NA][4], bh[MT][4], bl[PACK ? 1 : MT][4];
    };
    // Up to 16 batch rows block b begins b steps into K and wraps around: started together at the same column, the
    // blocks would ask the same few memory channels at the same time all along K (201 MB read this way and nothing
    // else: 38.1 us from a common first column, 32.5 from rotated ones).  Where a row is a multiple of 4 KB, so that all
    // rows begin on the same channels, the kernels of K = 2048, 4096, 6144, 8192 gained 5, 8, 8 and 9 % on average over 4, 6
    // and 16 rows; other lengths are within 3 % (K = 11008 and 22016 gained 2 and 10, 9472 lost 3).  4-bit rows are a
    // quarter as long: rotation cost 1 % on average, whole step of the 8B shape at 4 rows 605 -> 613 us, and paid at
    // K = 8192 only (rows of 4 KB; layers of 8192 x 22016, 4 rows 506 -> 497).  Rows off the 128 grid lost (layers of
    // 4104 x 11000, 16 rows 1310 -> 1362).  Beyond 16 rows, and where groups of rows share the weights through the caches,
    // the stream is not the limit.
    const int rot = MT == 1 && KALIGNED && (!Q4 || K % 8192 == 0) && gridDim.y == 1 ? (int)blockIdx.x % nks : 0;
    auto step = [&](int it) { const int ks = min(it * KS + wv, nks - 1) + rot; return ks < nks ? ks : ks - nks; };
    int it_i = 0;   // step to issue next
    auto issue = [&](Stage &st) {
        const int g = (int)blockIdx.x;
        const int ks = step(it_i);
        const int kb = ks * 128 + lg * 8;
        if constexpr (Q4) {
            const int n_tiles16 = (N + 15) >> 4;
#pragma unroll
            for (int m = 0; m < NA; m++) {
                const uint8_t *base = reinterpret_cast<const uint8_t *>((m / RT) ? a.W2 : a.W);
                const int tile = min(g * RT + (m % RT), n_tiles16 - 1);
                const int wrow = min(tile * 16 + ln, N - 1);
                st.wa[m][0] = ld16(base + (int64_t)wrow * (K >> 1) + ks * 64 + lg * 16);
                const uint8_t *sb = base + (int64_t)N * (K >> 1) + (((int64_t)tile * nks + ks) * 4 + lg) * 32;
                st.wa[m][1] = ld16(sb);
                st.wa[m][2] = ld16(sb + 16);
            }
            const int64_t xb = ((int64_t)ks * 4 * 64 + lane) * 8;
#pragma unroll
            for (int s = 0; s < 4; s++)
#pragma unroll
                for (int t = 0; t < MT; t++) {
                    const int64_t xo = xb + ((int64_t)t * nks * 4 + s) * 512;
                    st.bh[t][s] = ld16(a.xhi + xo);
                    if (!PACK) st.bl[t][s] = ld16(a.xlo + xo);
                }
            it_i++;
            return;
        }
        const uint16_t *wq[NA];
#pragma unroll
        for (int m = 0; m < NA; m++) {
            // tile m: matrix m / RT, rows of group g; rows past the end are clamped
            const int wrow = min(g * (16 * RT) + 16 * (m % RT) + ln, N - 1);
            wq[m] = ((m / RT) ? a.W2 : a.W) + (int64_t)wrow * K + kb;
        }
        const int64_t xb = ((int64_t)ks * 4 * 64 + lane) * 8;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            // aligned K: constant offsets; otherwise clamped into the row
            const int ko = KALIGNED ? s * 32 : min(kb + s * 32, K - 8) - kb;
#pragma unroll
            for (int m = 0; m < NA; m++) st.wa[m][s] = ld16(wq[m] + ko);
#pragma unroll
            for (int t = 0; t < MT; t++) {
                const int64_t xo = xb + ((int64_t)t * nks * 4 + s) * 512;
                st.bh[t][s] = ld16(a.xhi + xo);
                if (!PACK) st.bl[t][s] = ld16(a.xlo + xo);
            }
        }
        it_i++;
    };
    auto consume = [&](Stage &st, int it) {
        if (it * KS + wv >= nks) return;   // a padding step of this wave (uniform branch)
        const int ks = step(it);
        if constexpr (Q4) {
            const uint4 one4 = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);
            const f32x4_t zero = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int h = 0; h < 2; h++) {
                // group sums of x for this lane's batch row (the same in all four accumulator rows)
                f32x4_t S[MT];
#pragma unroll
                for (int t = 0; t < MT; t++) {
                    S[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(one4), as_bf16x8(st.bh[t][2 * h]), zero, 0, 0, 0);
                    if (!PACK) S[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(one4), as_bf16x8(st.bl[t][2 * h]), S[t], 0, 0, 0);
                    S[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(one4), as_bf16x8(st.bh[t][2 * h + 1]), S[t], 0, 0, 0);
                    if (!PACK) S[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(one4), as_bf16x8(st.bl[t][2 * h + 1]), S[t], 0, 0, 0);
                }
#pragma unroll
                for (int m = 0; m < NA; m++) {
                    const uint4 sb = st.wa[m][1 + h];
                    const uint32_t sbw[4] = {sb.x, sb.y, sb.z, sb.w};
                    float sc[4], b2[4];
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        sc[i] = __uint_as_float(sbw[i] << 16);
                        b2[i] = __uint_as_float(sbw[i] & 0xFFFF0000u);
                    }
                    const uint4 a0 = q4_codes_bf16(h ? st.wa[m][0].z : st.wa[m][0].x);
                    const uint4 a1 = q4_codes_bf16(h ? st.wa[m][0].w : st.wa[m][0].y);
#pragma unroll
                    for (int t = 0; t < MT; t++) {
                        f32x4_t D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a0), as_bf16x8(st.bh[t][2 * h]), zero, 0, 0, 0);
                        if (!PACK) D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a0), as_bf16x8(st.bl[t][2 * h]), D, 0, 0, 0);
                        D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a1), as_bf16x8(st.bh[t][2 * h + 1]), D, 0, 0, 0);
                        if (!PACK) D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a1), as_bf16x8(st.bl[t][2 * h + 1]), D, 0, 0, 0);
#pragma unroll
                        for (int i = 0; i < 4; i++)
                            acc[m][t][i] = fmaf(sc[i], D[i], fmaf(b2[i], S[t][i], acc[m][t][i]));
                    }
                }
            }
            return;
        }
        if constexpr (PACK == 3) {
            // A step's sum on its own, then onto the total: half the rounding error of one long chain in the matrix
            // cores, and below that of the vector kernel (relative error of logits against float64, K = 1024 / 4096 / 12288:
            // 0.9 / 1.1 / 1.3e-7; vector kernel 0.9 / 1.2 / 1.5e-7; one chain of products alone 1.0 / 1.9 / 3.3e-7).
#pragma unroll
            for (int m = 0; m < NA; m++) {
                f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; s++)
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(st.wa[m][s]), as_bf16x8(st.bh[0][s]), d, 0, 0, 0);
                acc[m][0] += d;
            }
        } else if constexpr (KALIGNED) {
#pragma unroll
            for (int s = 0; s < 4; s++)
#pragma unroll
                for (int t = 0; t < MT; t++)
#pragma unroll
                    for (int m = 0; m < NA; m++) {
                        acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            as_bf16x8(st.wa[m][s]), as_bf16x8(st.bh[t][s]), acc[m][t], 0, 0, 0);
                        if (!PACK)
                            acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                as_bf16x8(st.wa[m][s]), as_bf16x8(st.bl[t][s]), acc[m][t], 0, 0, 0);
                    }
        } else if constexpr (!KALIGNED) {
            const int kb = ks * 128 + lg * 8;
#pragma unroll
            for (int s = 0; s < 4; s++) {
                // past the end of K both operands are zeroed (the padding of the
                // activation buffer is not initialised)
                const bool in = kb + s * 32 < K;
                const uint4 z = make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int t = 0; t < MT; t++) {
                    const uint4 h4 = in ? st.bh[t][s] : z, l4 = in ? st.bl[t][s] : z;
#pragma unroll
                    for (int m = 0; m < NA; m++) {
                        const uint4 w4 = in ? st.wa[m][s] : z;
                        acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w4), as_bf16x8(h4),
                                                                            acc[m][t], 0, 0, 0);
                        acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w4), as_bf16x8(l4),
                                                                            acc[m][t], 0, 0, 0);
                    }
                }
            }
        }
    };

    // Sum-of-squares partials of the input rows: requested before the weight
    // stream starts and added up while its first stages are under way.
    SsqPartials<MT, KS> ssq;
    if (NORM) ssq.request(a.ssq_in, a.n_part, wv, lane);

    // The residual rows and the next norm's gains that the epilogue of wave rt < RT will
    // need: requested ahead of the weight stream as well (clamped addresses; used only
    // where valid), so that the epilogue does not end on a memory round trip.
    float xr[MT][4], gn[4];
    if (EPI == GEPI_RESID) {
        const int rr = ((int)blockIdx.x * RT + min(wv, RT - 1)) * 16 + 4 * lg;
#pragma unroll
        for (int i = 0; i < 4; i++) gn[i] = bf16_to_f32(a.gain_next[min(rr + i, N - 1)]);
#pragma unroll
        for (int t = 0; t < MT; t++) load_resid4(a.xres + (int64_t)min(t * 16 + ln, a.B - 1) * N, rr, N, xr[t]);
    }

    Stage st[PD];
#pragma unroll
    for (int p = 0; p < PD; p++) issue(st[p]);
    if (NORM) ssq.store(a.ssq_in, a.n_part, wv, lane, ssq_s[wv]);   // while the first weights are under way

    {
        for (int it = 0; it + PD < niter2; it += PD) {
#pragma unroll
            for (int p = 0; p < PD; p++) {
                consume(st[p], it + p);
                issue(st[p]);
            }
        }
#pragma unroll
        for (int p = 0; p < PD; p++) consume(st[p], niter2 - PD + p);
        // K-splits meet in LDS
        RedBuf &rb = red[0];
#pragma unroll
        for (int m = 0; m < NA; m++)
#pragma unroll
            for (int t = 0; t < MT; t++)
#pragma unroll
                for (int i = 0; i < 4; i++) rb[wv][m][t][i][lane] = acc[m][t][i];
        __syncthreads();
        if (wv >= RT) return;

        // Wave rt < RT finishes row tile rt of the group: it adds the K-splits in
        // wave order, then the epilogue.  The lane holds
        // D[row0 + 4*lg + i][n = 16*t + ln], i = 0..3.
        const int rt = wv;
        const int out_tile = (int)blockIdx.x * RT + rt;
        if (out_tile * 16 >= N) return;
        float v[MT][NM][4];
#pragma unroll
        for (int t = 0; t < MT; t++) {
            const int n = t * 16 + ln;
#pragma unroll
            for (int m = 0; m < NM; m++)
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    float s = 0.f;
#pragma unroll
                    for (int w = 0; w < KS; w++) s += rb[w][m * RT + rt][t][i][lane];
                    v[t][m][i] = pack_sum<PACK>(s, lane);
                }
            if (NORM) {
                float s = 0.f;
#pragma unroll
                for (int w = 0; w < KS; w++) s += ssq_s[w][n];
                const float inv = rsqrtf(s / (float)K + a.eps);
#pragma unroll
                for (int m = 0; m < NM; m++)
#pragma unroll
                    for (int i = 0; i < 4; i++) v[t][m][i] *= inv;
            }
        }
        gemm_tile_epilogue<MT, EPI, PACK>(a, out_tile, lane, v, xr, gn);
    }
}

// Dynamic LDS bytes of a skinny_gemm_kernel instance.
template <int MT, int KS, int RT, int EPI>
constexpr size_t skinny_gemm_lds_bytes()
{
    return (size_t)KS * ((EPI == GEPI_SWIGLU) ? 2 : 1) * RT * MT * 4 * 64 * 4 + (size_t)KS * 64 * 4;
}

}  // namespace dk
