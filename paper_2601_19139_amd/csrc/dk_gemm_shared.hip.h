// Skinny GEMM whose waves share one activation tile.
//
// Same contract and epilogues as skinny_gemm_kernel (dk_gemm.hip.h).  There every wave of a block
// takes other K-steps, so every wave fetches its own activation operands: 8 KB of bf16 hi/lo
// per 128-column step and 16 batch rows, against 4 KB of weights per row tile.  At 32..64 rows that
// is 4..8 times the weight stream and bounds the kernel; up to 16 rows it matters where a wave has
// one row tile or the stream is long.  Here all W waves of a block walk the SAME
// K-steps and own different row tiles: the block fetches each step's activation tile once,
// 16 bytes per thread, puts it into LDS, and every wave reads its matrix-core operands from
// there.  A wave then carries only weights (and its 16-byte share of the activations) in
// flight, so the software pipeline can be deeper for the same registers, and a tile's sum over
// K is complete in one wave - no reduction across waves.
//
// The price is a barrier per K-step, which couples the waves of a block to its slowest load.  Measured
// on the 8B / 3B / 0.6B shapes this pays above 16 rows for the lm_head (2-3.5x) and for the large layer
// matrices from 33 rows on (1.2-1.6x); up to 16 rows for the lm_head, long residual projections and the
// gate/up pairs of more than two row tiles per compute unit (both sides at gemm_plan_16) - the host picks.
//
// A matrix with few row tiles would leave compute units idle, so K can be cut into gridDim.y
// slices.  Each block then stores its partial tiles (device-coherent stores: the dies' L2s
// are not coherent with each other), takes a ticket of its row block, and the block that
// arrives last adds the slices in slice order and runs the epilogue: the result does not
// depend on arrival order.
#pragma once
#include "dk_attention.hip.h"
#include "dk_gemm.hip.h"

namespace dk {

// Floats of partial tiles a K-sliced GEMM needs: [slice][matrix][tile][column tile][64 lanes][4].
__host__ __device__ inline size_t shared_gemm_part_floats(int N, int slices, int n_mat, int MT)
{
    return (size_t)slices * n_mat * ((N + 15) / 16) * MT * 256;
}

// Device-scope 16-byte accesses (raw buffer instructions with the sc1 bit) at base + byte_off, the words of one
// lane's partial tile.  base: uniform over the wave, 16-byte aligned; bytes: the extent reachable from base.
// The scalar atomics they replace moved 4 bytes per lane and instruction: a quarter of the requests for the
// hand-over of a slice, on the way out and on the way back (501-token prefill of the 8B shape 49.1 -> 48.7 ms).
__device__ __forceinline__ void st_coherent16(float *base, int bytes, uint32_t byte_off, const f32x4_t &v)
{
    typedef uint32_t words_t __attribute__((ext_vector_type(4)));
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(words_t, v), rsrc, (int)byte_off, 0, 16);
}
__device__ __forceinline__ f32x4_t ld_coherent16(const float *base, int bytes, uint32_t byte_off)
{
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, bytes, 0x00020000);
    return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)byte_off, 0, 16));
}

// Dynamic LDS bytes of a shared_gemm_kernel instance.
constexpr size_t shared_gemm_lds_bytes(int MT) { return (size_t)2 * 512 * MT * 16; }

// A block's 128 output rows are one head of k or v of a prompt chunk: head norm and rotation (k), rounding, and into the
// pool, as prefill_append_kernel does it (same arithmetic).  That kernel is a launch of its own, 4.9 us per layer, for
// values that this block has in its registers; here the head takes one trip through the LDS of the activation tiles and
// the projection 0.3 us more at the 8B shape (64 rows, 23.9 -> 24.2), 0.9 at the 3B shape with 4-bit weights (19.4 -> 20.3).
// buf: [rows][132] floats.  Called by all threads, which have left the activation tiles.
template <int MT, int W>
__device__ __forceinline__ void append_head(const GemmArgs &a, int head, const float (&v)[MT][4], float *buf)
{
    constexpr int D = 128, BS = 16, LD = D + 4;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, ln = lane & 15, lg = lane >> 4;
#pragma unroll
    for (int t = 0; t < MT; t++)
        *reinterpret_cast<float4 *>(buf + (t * 16 + ln) * LD + wv * 16 + 4 * lg) = make_float4(v[t][0], v[t][1], v[t][2], v[t][3]);
    __syncthreads();
    const bool is_v = head >= a.kv_heads;
    const int j = is_v ? head - a.kv_heads : head, dl = (tid & 15) * 8;
    const bool upper = dl >= D / 2, norm = a.g_k != nullptr;
    float gk[8];
    if (norm) {
        unpack8(ld16(a.g_k + dl), gk);
    } else {
#pragma unroll
        for (int e = 0; e < 8; e++) gk[e] = 1.f;
    }
    for (int n = tid >> 4; n < a.B; n += W * 4) {   // sixteen lanes to a row
        const int T = min(max(a.seq_lens[n], 0), a.max_blocks * BS - 1);
        const int phys = min(max(a.block_table[T / BS], 0), a.num_blocks - 1);
        const float4 lo = ldf4(buf + n * LD + dl), hi = ldf4(buf + n * LD + dl + 4);
        float x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        if (!is_v) {
            float2 cs[8];
            const float4 *cp = reinterpret_cast<const float4 *>(a.cs + (int64_t)n * (D / 2) + (upper ? dl - D / 2 : dl));
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const float4 t = cp[e];
                cs[2 * e] = make_float2(t.x, t.y);
                cs[2 * e + 1] = make_float2(t.z, t.w);
            }
            head_norm_rope<D>(x, norm, gk, a.eps, cs, upper);
        }
        uint16_t *dst = a.pool + kv_tile_offset(a.layer, a.num_blocks, phys, is_v ? 1 : 0, a.kv_heads, j, BS, D) + (T % BS) * D + dl;
        *reinterpret_cast<uint4 *>(dst) = make_uint4(f32x2_to_bf16x2_rne(x[0], x[1]), f32x2_to_bf16x2_rne(x[2], x[3]),
                                                     f32x2_to_bf16x2_rne(x[4], x[5]), f32x2_to_bf16x2_rne(x[6], x[7]));
    }
}

// W waves per block, RT row tiles per wave (GEPI_SWIGLU: of each of the two matrices), PD K-steps
// in flight per wave.  K must be a multiple of 128.  grid = (ceil(tiles / (W*RT)), slices).
// Q4: packed 4-bit weights, evaluated as in skinny_gemm_kernel's Q4 variant (codes through the matrix
// cores, group sums of x from an all-ones operand, scale and bias applied to the fp32 tiles).
// PACK (MT = 1): xhi is one operand with PACK terms of every row, half of the pieces (both halves of an 8-wave block fetch them).
template <int MT, int W, int RT, int PD, int EPI, bool NORM, bool Q4 = false, int PACK = 0>
__global__ __launch_bounds__(W * 64) void shared_gemm_kernel(GemmArgs a)
{
    constexpr int NM = (EPI == GEPI_SWIGLU) ? 2 : 1;
    constexpr int NA = NM * RT;
    constexpr int TPB = W * 64;
    constexpr int PIECES = PACK ? 256 : 512 * MT;   // 16-byte pieces of one step's activation tile (hi and lo)
    static_assert(PACK == 0 || (MT == 1 && TPB % 256 == 0), "a packed tile is 256 pieces");
    constexpr int PPT = PACK ? 1 : (PIECES + TPB - 1) / TPB;   // (six waves: the last round is one of whole waves)
    constexpr int NC = W == 6 ? 8 : W;                         // classes of the sum-of-squares partials: as with eight waves
    extern __shared__ uint4 sm_act_dyn[];   // two slots of one step's activation tile (shared_gemm_lds_bytes)
    uint4 (*sm_act)[PIECES] = reinterpret_cast<uint4 (*)[PIECES]>(sm_act_dyn);
    __shared__ __align__(16) float sm_ssq[NC][64];
    __shared__ int sm_last;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ln = lane & 15, lg = lane >> 4;
    const int K = a.K, N = a.N;
    const int nks = K >> 7, n_tiles = (N + 15) >> 4;
    const int S = (int)gridDim.y, y = (int)blockIdx.y;
    const int ks0 = (int)((long long)nks * y / S), ks1 = (int)((long long)nks * (y + 1) / S);
    const int niter = ks1 - ks0;
    const int niter2 = (niter + PD - 1) / PD * PD;
    const int tile0 = ((int)blockIdx.x * W + wv) * RT;

    f32x4_t acc[NA][MT];
#pragma unroll
    for (int m = 0; m < NA; m++)
#pragma unroll
        for (int t = 0; t < MT; t++) acc[m][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Same pipeline discipline as skinny_gemm_kernel: no conditional loads, every wave runs a
    // multiple of PD steps, steps past the slice read clamped addresses and are not used.
    struct Stage {
        uint4 wa[NA][Q4 ? 3 : 4], act[PPT];   // Q4: codes of the whole step, (scale, bias) of its two groups
    };
    // Where a block begins in its slice.  Up to 16 rows every block at another column (see skinny_gemm_kernel).  Above, in
    // the gate/up pair of a decode step (a.spread), the blocks of a compute die together, since they share the activation
    // tiles of a step through its L2, and the dies an eighth of the slice apart: with all blocks at one column of rows
    // 8 KB apart their weights come from a few memory channels (12288 x 4096: 64 rows 55.2 -> 51.7 us, 32 rows 50.3 ->
    // 40.7; 8192 x 3072 30.9 -> 30.1; the other matrices and 4-bit rows the same as before).  Not for prompts: their K/V,
    // rounded to bf16, feed all that follows, so there another order of sums shows as 1e-3 of the logits.
    int rot = 0;
    if (MT == 1) rot = !Q4 || K % 8192 == 0 ? (int)blockIdx.x % max(niter, 1) : 0;
    else if (EPI == GEPI_SWIGLU && !Q4 && a.spread) rot = (int)((blockIdx.x + blockIdx.y * gridDim.x) & 7) * niter / 8;
    int it_i = 0;
    auto issue = [&](Stage &st) {
        // (a step past the slice, or an empty slice - more slices than steps: a valid step, unused)
        int ks = max(min(it_i, niter - 1), 0) + rot;
        ks = min(ks0 + (ks < niter ? ks : ks - niter), nks - 1);
#pragma unroll
        for (int p = 0; p < PPT; p++) {
            const int piece = PACK ? (tid & 255) : PIECES % TPB ? min(p * TPB + tid, PIECES - 1) : p * TPB + tid;
            const int t = piece >> 9, lo = (piece >> 8) & 1, idx = piece & 255;
            st.act[p] = ld16((lo ? a.xlo : a.xhi) + (((int64_t)t * nks + ks) * 256 + idx) * 8);
        }
#pragma unroll
        for (int m = 0; m < NA; m++) {
            if constexpr (Q4) {
                const uint8_t *base = reinterpret_cast<const uint8_t *>((m / RT) ? a.W2 : a.W);
                const int tile = min(tile0 + (m % RT), n_tiles - 1);
                const int wrow = min(tile * 16 + ln, N - 1);
                st.wa[m][0] = ld16(base + (int64_t)wrow * (K >> 1) + ks * 64 + lg * 16);
                const uint8_t *sb = base + (int64_t)N * (K >> 1) + (((int64_t)tile * nks + ks) * 4 + lg) * 32;
                st.wa[m][1] = ld16(sb);
                st.wa[m][2] = ld16(sb + 16);
            } else {
                const int wrow = min((tile0 + (m % RT)) * 16 + ln, N - 1);   // rows past the end are clamped
                const uint16_t *wq = ((m / RT) ? a.W2 : a.W) + (int64_t)wrow * K + ks * 128 + lg * 8;
#pragma unroll
                for (int s = 0; s < 4; s++) st.wa[m][s] = ld16(wq + s * 32);
            }
        }
        it_i++;
    };
    auto consume = [&](Stage &st, int it) {
        if (it < 0 || it >= niter) return;   // a padding step (the same for the whole block)
        uint4 *slot = sm_act[it & 1];
#pragma unroll
        for (int p = 0; p < PPT; p++)
            if (PACK ? tid < 256 : (PIECES % TPB == 0 || p * TPB + tid < PIECES)) slot[p * TPB + tid] = st.act[p];
        // one barrier per step is enough with two slots: nobody can write this slot again
        // before every wave has passed the next step's barrier, i.e. has finished reading it
        __syncthreads();
        if constexpr (Q4) {
            const uint4 one4 = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);
            const f32x4_t zero = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int h = 0; h < 2; h++) {
                uint4 c0[NA], c1[NA];
                float sc[NA][4], bi[NA][4];
#pragma unroll
                for (int m = 0; m < NA; m++) {
                    c0[m] = q4_codes_bf16(h ? st.wa[m][0].z : st.wa[m][0].x);
                    c1[m] = q4_codes_bf16(h ? st.wa[m][0].w : st.wa[m][0].y);
                    const uint4 sb = st.wa[m][1 + h];
                    const uint32_t sbw[4] = {sb.x, sb.y, sb.z, sb.w};
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        sc[m][i] = __uint_as_float(sbw[i] << 16);
                        bi[m][i] = __uint_as_float(sbw[i] & 0xFFFF0000u);
                    }
                }
#pragma unroll
                for (int t = 0; t < MT; t++) {
                    constexpr int LO = PACK ? 0 : 256;   // (packed: the lo operand does not exist and is not used)
                    const uint4 bh0 = slot[t * 512 + (2 * h) * 64 + lane], bl0 = slot[t * 512 + LO + (2 * h) * 64 + lane];
                    const uint4 bh1 = slot[t * 512 + (2 * h + 1) * 64 + lane], bl1 = slot[t * 512 + LO + (2 * h + 1) * 64 + lane];
                    // group sums of x for this lane's batch row (the same in all four accumulator rows)
                    f32x4_t S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(one4), as_bf16x8(bh0), zero, 0, 0, 0);
                    if (!PACK) S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(one4), as_bf16x8(bl0), S, 0, 0, 0);
                    S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(one4), as_bf16x8(bh1), S, 0, 0, 0);
                    if (!PACK) S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(one4), as_bf16x8(bl1), S, 0, 0, 0);
#pragma unroll
                    for (int m = 0; m < NA; m++) {
                        f32x4_t D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(c0[m]), as_bf16x8(bh0), zero, 0, 0, 0);
                        if (!PACK) D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(c0[m]), as_bf16x8(bl0), D, 0, 0, 0);
                        D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(c1[m]), as_bf16x8(bh1), D, 0, 0, 0);
                        if (!PACK) D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(c1[m]), as_bf16x8(bl1), D, 0, 0, 0);
#pragma unroll
                        for (int i = 0; i < 4; i++)
                            acc[m][t][i] = fmaf(sc[m][i], D[i], fmaf(bi[m][i], S[i], acc[m][t][i]));
                    }
                }
            }
            return;
        }
        if constexpr (PACK == 3) {   // a step's sum on its own, then onto the total (see skinny_gemm_kernel)
#pragma unroll
            for (int m = 0; m < NA; m++) {
                f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < 4; s++)
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(st.wa[m][s]), as_bf16x8(slot[s * 64 + lane]), d, 0, 0, 0);
                acc[m][0] += d;
            }
            return;
        }
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
            for (int t = 0; t < MT; t++) {
                const uint4 bh = slot[t * 512 + s * 64 + lane], bl = slot[t * 512 + (PACK ? 0 : 256) + s * 64 + lane];
#pragma unroll
                for (int m = 0; m < NA; m++) {
                    acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(st.wa[m][s]), as_bf16x8(bh),
                                                                        acc[m][t], 0, 0, 0);
                    if (!PACK)
                        acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(st.wa[m][s]), as_bf16x8(bl),
                                                                            acc[m][t], 0, 0, 0);
                }
            }
    };

    // sum-of-squares partials of the input rows (NORM), requested ahead of the stream
    SsqPartials<MT, NC> ssq;
    if (NORM) ssq.request(a.ssq_in, a.n_part, wv, lane);
    // residual rows and next gains of this wave's tiles (GEPI_RESID)
    float xr[RT][MT][4], gn[RT][4];
    if (EPI == GEPI_RESID) {
#pragma unroll
        for (int r = 0; r < RT; r++) {
            const int rr = (tile0 + r) * 16 + 4 * lg;
#pragma unroll
            for (int i = 0; i < 4; i++) gn[r][i] = bf16_to_f32(a.gain_next[min(rr + i, N - 1)]);
#pragma unroll
            for (int t = 0; t < MT; t++) load_resid4(a.xres + (int64_t)min(t * 16 + ln, a.B - 1) * N, rr, N, xr[r][t]);
        }
    }

    Stage st[PD];
#pragma unroll
    for (int p = 0; p < PD; p++) issue(st[p]);
    if (NORM) ssq.store(a.ssq_in, a.n_part, wv, lane, sm_ssq[wv]);   // while the first weights are under way
    for (int it = 0; it + PD < niter2; it += PD) {
#pragma unroll
        for (int p = 0; p < PD; p++) {
            consume(st[p], it + p);
            issue(st[p]);
        }
    }
#pragma unroll
    for (int p = 0; p < PD; p++) consume(st[p], niter2 - PD + p);

    if (NORM && W < NC && wv + W < NC) {   // the classes without a wave of their own
        ssq.request(a.ssq_in, a.n_part, wv + W, lane);
        ssq.store(a.ssq_in, a.n_part, wv + W, lane, sm_ssq[wv + W]);
    }

    if (S > 1) {
        // partial tiles out, ticket, and only the last block of this row block goes on
        const size_t slice_floats = (size_t)NM * n_tiles * MT * 256;
#pragma unroll
        for (int m = 0; m < NA; m++) {
            const int tile = tile0 + (m % RT);
            if (tile >= n_tiles) continue;
            float *pp = a.kpart + (size_t)y * slice_floats + ((size_t)(m / RT) * n_tiles + tile) * MT * 256;
#pragma unroll
            for (int t = 0; t < MT; t++) st_coherent16(pp, MT * 1024, (uint32_t)(t * 1024 + lane * 16), acc[m][t]);
        }
        drain_stores();    // every wave's partial tiles are complete ...
        __syncthreads();   // ... before one thread takes the ticket
        if (tid == 0)
            sm_last = __hip_atomic_fetch_add(&a.ktickets[blockIdx.x], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                      S - 1;
        __syncthreads();
        if (!sm_last) return;
        if (tid == 0) __hip_atomic_store(&a.ktickets[blockIdx.x], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // Slices are added in slice order (the result does not depend on who arrived last).  The
        // device-coherent loads of a slice - 16 bytes per lane and 16 x 16 tile, as the matrix cores
        // leave it - are independent and are all issued before the first is used; the next slice is
        // requested before this one is added, so a round trip is paid per slice, not per element.
        // The block's own slice is still in its registers (with two slices half of the bytes that the last
        // blocks, a part of the chip, read alone: gate/up of 12288 x 4096, 64 rows, begun at columns apart, 51.7 -> 47.9 us).
        const float *pbase[NA];
#pragma unroll
        for (int m = 0; m < NA; m++) {
            const int tile = min(tile0 + (m % RT), n_tiles - 1);
            pbase[m] = a.kpart + ((size_t)(m / RT) * n_tiles + tile) * MT * 256;
        }
        auto fetch = [&](int q, f32x4_t (&v)[NA][MT]) {
            const size_t off = (size_t)min(q, S - 1) * slice_floats;
#pragma unroll
            for (int m = 0; m < NA; m++)
#pragma unroll
                for (int t = 0; t < MT; t++)
                    v[m][t] = ld_coherent16(pbase[m] + off, MT * 1024, (uint32_t)(t * 1024 + lane * 16));
        };
        f32x4_t own[NA][MT], cur[NA][MT], nxt[NA][MT];
        auto other = [&](int i) { return i + (i >= y ? 1 : 0); };   // the i-th of the other slices
        fetch(other(0), cur);
#pragma unroll
        for (int m = 0; m < NA; m++)
#pragma unroll
            for (int t = 0; t < MT; t++) {
                own[m][t] = acc[m][t];
                acc[m][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
        auto add = [&](const f32x4_t (&v)[NA][MT]) {
#pragma unroll
            for (int m = 0; m < NA; m++)
#pragma unroll
                for (int t = 0; t < MT; t++) acc[m][t] += v[m][t];
        };
        for (int i = 0; i < S - 1; i++) {
            fetch(other(i + 1), nxt);       // (past the last slice: the last one again, unused)
            if (i == y) add(own);
            add(cur);
#pragma unroll
            for (int m = 0; m < NA; m++)
#pragma unroll
                for (int t = 0; t < MT; t++) cur[m][t] = nxt[m][t];
        }
        if (y == S - 1) add(own);
    } else {
        __syncthreads();   // sm_ssq
    }

    float inv[MT];
#pragma unroll
    for (int t = 0; t < MT; t++) {
        inv[t] = 1.f;
        if (NORM) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < NC; w++) s += sm_ssq[w][t * 16 + ln];
            inv[t] = rsqrtf(s / (float)K + a.eps);
        }
    }
    if constexpr (EPI == GEPI_STORE && W == 8 && RT == 1) {
        if (a.q_heads > 0 && (int)blockIdx.x >= a.q_heads) {
            float v[MT][4];
#pragma unroll
            for (int t = 0; t < MT; t++)
#pragma unroll
                for (int i = 0; i < 4; i++) v[t][i] = pack_sum<PACK>(acc[0][t][i], lane) * inv[t];
            append_head<MT, W>(a, (int)blockIdx.x - a.q_heads, v, reinterpret_cast<float *>(sm_act_dyn));
            return;
        }
    }
#pragma unroll
    for (int r = 0; r < RT; r++) {
        const int tile = tile0 + r;
        if (tile >= n_tiles) continue;
        float v[MT][NM][4];
#pragma unroll
        for (int t = 0; t < MT; t++)
#pragma unroll
            for (int m = 0; m < NM; m++)
#pragma unroll
                for (int i = 0; i < 4; i++) v[t][m][i] = pack_sum<PACK>(acc[m * RT + r][t][i], lane) * inv[t];
        gemm_tile_epilogue<MT, EPI, PACK>(a, tile, lane, v, xr[r], gn[r]);
    }
}

}  // namespace dk
