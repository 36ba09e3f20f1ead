// HIP kernels of the block-decode step for gfx950 (CDNA4).
//
// One forward pass over a k-token block per sequence (arXiv 2607.05722,
// Sec. 3.3, linear self-speculation) is:
//   embed -> L x [QKV GEMM (RMSNorm fused into the operand load; RoPE and the
//                 K/V cache write fused into the epilogue),
//                 block-masked GQA attention over key splits (+ split merge),
//                 O GEMM (+ residual),
//                 gate/up GEMM (RMSNorm fused; SwiGLU epilogue),
//                 down GEMM (+ residual)]
//         -> LM-head GEMM (final RMSNorm fused; per-workgroup argmax keys)
//         -> per-sequence argmax + draft extraction / acceptance.
//
// The GEMMs are skinny (M = batch*k rows, from one to a few hundred): up to about a
// hundred rows they are bound by streaming the bf16 weights from HBM.  Weights are pre-packed so that one 16-byte load per
// lane of a wavefront is exactly one MFMA B operand (1 KiB contiguous per
// wavefront load).
//
// Communication between workgroups of one launch.  The normed GEMM hands out
// tiles from a counter.  The split-K GEMM and the panel GEMM with K slices meet
// through last-arriver counters; no workgroup ever waits for another.  The protocol
// of a slice partial:
//   1. every lane writes its part with agent-scope stores (relaxed atomics, or
//      16-byte buffer stores with the same cache bits);
//   2. s_waitcnt(0): the wavefront waits until each of its stores is
//      acknowledged, then a workgroup barrier;
//   3. one thread adds 1 to the counter (agent-scope relaxed fetch_add); the
//      workgroup that reads ksplit - 1 is the last to arrive;
//   4. the last arriver resets the counter to 0, reads the other partials with
//      agent-scope loads, adds the slices in slice order (so the
//      sum does not depend on who arrived last) and runs the epilogue.
// Why this orders the data: agent-scope stores are made visible at agent scope
// (past the XCD-local L2) by the time they are acknowledged, so after step 2
// the partials are readable by agent-scope loads from any XCD; the barrier and
// the data dependence through the counter's value order step 4 after step 3.
// The C++ memory model would ask for an agent-scope release fence before the
// fetch_add (an L2 write-back measured at 11-18 us per kernel here); relaxed
// stores plus the store-acknowledgement wait rely instead on how gfx950
// completes agent-scope stores.  Repeated passes giving bit-identical results
// guard it in the tests.  Every counter is back at zero when its kernel ends,
// and the embedding kernel zeroes all of them at the start of each pass.

#include "nld_internal.h"

#include <hip/hip_ext.h>

#include <math.h>

namespace nld {

// Per-workgroup phase timestamps (a diagnostic build only, -DNLD_TIMELINE; see timeline.py): thread 0
// of each workgroup records the 100 MHz real-time counter at the phase boundaries of the kernels of
// one layer pass, class x workgroup x phase.  In the normal build NLD_TS expands to nothing.
#ifdef NLD_TIMELINE
__device__ unsigned long long g_timeline[8][8192][8];
#define NLD_TS(cls, ph)                                                                                   \
    do {                                                                                                  \
        if (threadIdx.x == 0)                                                                             \
            g_timeline[cls][blockIdx.x + blockIdx.y * gridDim.x + blockIdx.z * gridDim.x * gridDim.y][ph] = \
                __builtin_amdgcn_s_memrealtime();                                                         \
    } while (0)
#else
#define NLD_TS(cls, ph) do { } while (0)
#endif
enum TimelineClass { TL_QKV = 0, TL_ATTENTION = 1, TL_COMBINE = 2, TL_GATE_UP = 3, TL_O = 4, TL_DOWN = 5, TL_LM = 6 };

// Every kernel launch goes through here: a plain launch, or, while launch tracing is on,
// a launch whose start and stop events are recorded on the dispatch itself.
template <typename... KArgs, typename... Args>
static void launch(void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t s, Args... args) {
    hipEvent_t e0, e1;
    if (trace_launch_events(&e0, &e1)) hipExtLaunchKernelGGL(kernel, grid, block, 0, s, e0, e1, 0, args...);
    else kernel<<<grid, block, 0, s>>>(args...);
}


static constexpr uint32_t DEV_BAD_TOKEN = 0x1u;
static constexpr uint32_t DEV_CAPACITY = 0x2u;
static constexpr uint32_t DEV_BAD_LENGTH = 0x4u;
static constexpr uint32_t DEV_MASK_LEFT = 0x8u;

__device__ __forceinline__ int committed_length(const int32_t* lengths, int b, int max_len, uint32_t* status) {
    int p = lengths[b];
    if (p < 0) {
        atomicOr(status, DEV_BAD_LENGTH);
        p = 0;
    }
    return p < max_len ? p : max_len;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

__device__ __forceinline__ unsigned long long umax64(unsigned long long a, unsigned long long b) { return a > b ? a : b; }

// =====================================================================================
// GEMM epilogues, one output row per call.  A 16x16 output tile (packed column tile
// t) is finished by up to four wavefronts together: the wavefront that takes index i
// handles rows 4g + i of the tile (g = lane / 16) and lane 16g + r holds column r.
// y is the finished (RMSNorm-scaled) value of row m, column r.
// =====================================================================================
// Softmax statistics as (max, sum of exp(z - max)); (-inf, 0) is the empty set.
__device__ __forceinline__ float2 lse_merge(float2 a, float2 b) {
    if (b.x == -INFINITY) return a;
    if (a.x == -INFINITY) return b;
    const float mx = fmaxf(a.x, b.x);
    return float2{mx, a.y * expf(a.x - mx) + b.y * expf(b.x - mx)};
}

// Returns, in every lane, the argmax key of row m over this tile's 16 columns and,
// when the pass asks for softmax statistics, the tile row's (max, sum of exp) in
// *lse.  The excluded column (the mask token when denoising) takes part in neither.
__device__ __forceinline__ unsigned long long epi_lmhead(const GemmArgs& a, float y, int m, int t, int lane,
                                                         float2* lse) {
    const int r = lane & 15;
    const int n = t * 16 + r;
    const bool in = m < a.M && n < a.vocab;
    const bool ok = in && n != a.exclude_id;
    if (in && a.logits) a.logits[(size_t)m * a.vocab + n] = y;
    if (in && a.ens_logits) {   // quadratic layout: the verifier rows (chain row i, mask 1 of group i)
        const int b = m / a.k_blk, jb = m - b * a.k_blk, qk = a.quad_k;
        const int ci = jb < qk ? jb : ((jb - qk) % qk == 0 ? qk + (jb - qk) / qk : -1);
        if (ci >= 0) a.ens_logits[((size_t)b * 2 * qk + ci) * a.vocab + n] = y;
    }
    unsigned long long key = ok ? argmax_key(y, (uint32_t)n) : 0ull;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) key = umax64(key, __shfl_xor(key, off));
    if (a.part_lse) {
        float mx = ok ? y : -INFINITY;
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        float e = ok ? expf(y - mx) : 0.f;
#pragma unroll
        for (int off = 1; off < 16; off <<= 1) e += __shfl_xor(e, off);
        *lse = float2{mx, e};
    }
    return key;
}

// xres: the residual x[m][16t + r]; gn: the next RMSNorm's gain at column 16t + r.
// Writes x += v, the next RMSNorm's split operand x * gain_next and the row's sum of
// x^2 over the tile's 16 columns.
__device__ __forceinline__ void epi_resid(const GemmArgs& a, float v, int m, int t, int lane, float xres, float gn) {
    const int r = lane & 15;
    const int N = a.n_tiles * 16;
    const int n = t * 16 + r;
    const bool ok = m < a.M;
    const float xn = xres + v;
    if (ok) {
        a.x[(size_t)m * N + n] = xn;
        store_split(a.xg_out, split_index(m, n, N / 32), xn * gn, a.plain & (SITE_NORM | SITE_FINAL));
    }
    float sq = ok ? xn * xn : 0.f;
    sq += __shfl_xor(sq, 1);
    sq += __shfl_xor(sq, 2);
    sq += __shfl_xor(sq, 4);
    sq += __shfl_xor(sq, 8);
    if (r == 0 && ok) a.part_ss_out[(size_t)m * a.n_tiles + t] = sq;
}

// 1/rms for `rows` rows starting at m0 from the producer's 16-column partial sums
// (fixed summation order); rows past M get 0.  One wavefront per row.
__device__ __forceinline__ void rms_scales(const GemmArgs& a, int m0, int rows, float* inv_s) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    for (int rr = wave; rr < rows; rr += nw) {
        const int m = m0 + rr;
        float s = 0.f;
        if (m < a.M) {
            const float* ps = a.part_ss + (size_t)m * a.n_ss;
            for (int p = lane; p < a.n_ss; p += 64) s += ps[p];
        }
        s = wave_sum(s);
        if (lane == 0) inv_s[rr] = (m < a.M) ? 1.0f / sqrtf(s / (float)a.K + a.eps) : 0.f;
    }
}

// =====================================================================================
// Normed multi-tile GEMM: the LM head of up to 16 rows.  A workgroup of NW wavefronts takes output tiles
// from a counter; wavefront w owns the reduction slice [32*KS*w, 32*KS*(w+1)).  At the start each wavefront
// loads its slice of the split operand bf16(x * gain) (hi and lo) and keeps it in registers for all tiles;
// the per-row RMSNorm scale comes from the producer's partial sums of squares.  Weights stream through one
// register buffer: the load of the next tile's step s is issued as soon as step s of the current tile has
// been multiplied, so one tile's worth of loads is in flight throughout.  Per tile the NW partial products
// meet in LDS and one group of wavefronts (rotating) runs the epilogue.  Against the panel GEMM it has no
// prologue per tile and no uneven last round, but only a full workgroup of full slices streams as fast: the rule of
// its dispatch has both sides' times.
// =====================================================================================
template <int NW, int KS>
__global__ void __launch_bounds__(NW * 64) gemm_norm_kernel(GemmArgs a) {
    __shared__ f32x4_t red[2][NW][64];
    __shared__ float inv_s[16];
    __shared__ unsigned long long key_s[NW][16];
    __shared__ float2 lse_s[NW][16];
    __shared__ int next_s[2];

    NLD_TS(TL_LM, 0);
    if (threadIdx.x < NW * 16) {
        key_s[threadIdx.x >> 4][threadIdx.x & 15] = 0ull;
        lse_s[threadIdx.x >> 4][threadIdx.x & 15] = float2{-INFINITY, 0.f};
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int T = a.n_tiles, G = gridDim.x;
    const int s0 = wave * KS;

    // Tiles are handed out dynamically: workgroup b starts with tile b, further tiles
    // come from a counter (tile index G + counter), requested one tile ahead so that
    // the atomic's latency hides behind the current tile.  Faster workgroups (and
    // XCDs) end up with more tiles.
    int cur = blockIdx.x;
    unsigned grab = 0u;
    if (threadIdx.x == 0 && G < T) grab = atomicAdd(a.tile_ctr, 1u);

    // operand slice: row r, columns 32*(s0+s) + 8g .. +8, hi and lo.  Requested before the first
    // weight tile: loads complete in issue order, and the operand (L2 hits after the first workgroups)
    // then no longer waits behind the tile's HBM reads (8B shapes, k = 16: 198.5 against 200.5 us).
    uint4 ah[KS], al[KS];
    const bool row_ok = r < a.M;
    const uint16_t* ar = a.A + (size_t)s0 * 1024 + (size_t)lane * 8;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        ah[s] = row_ok ? *(const uint4*)(ar + (size_t)s * 1024) : uint4{0u, 0u, 0u, 0u};
        al[s] = row_ok ? *(const uint4*)(ar + (size_t)s * 1024 + SPLIT_LO) : uint4{0u, 0u, 0u, 0u};
    }
    uint4 wb[KS];
    if (cur < T) {
        const uint4* p = a.W + ((size_t)cur * a.ksteps + s0) * 64 + lane;
#pragma unroll
        for (int s = 0; s < KS; ++s) wb[s] = load_stream(p + (size_t)s * 64);
    }
    rms_scales(a, 0, 16, inv_s);
    if (threadIdx.x == 0) next_s[0] = G < T ? min(G + (int)grab, T) : T;
    __syncthreads();

    // A tile is finished by FIN wavefronts (wavefront i of the group takes rows 4g + i); the groups take the tiles in turn.
    NLD_TS(TL_LM, 1);   // operand, first tile and row statistics in
    constexpr int FIN = 4, groups = NW / FIN;
    for (int it = 0; cur < T; ++it) {
        const int t = cur;
        const int nxt = next_s[it & 1];   // its weights stream in while tile t is multiplied
        if (threadIdx.x == 0 && nxt < T) grab = atomicAdd(a.tile_ctr, 1u);
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f}, accl = {0.f, 0.f, 0.f, 0.f};
        const bool more = nxt < T;
        const uint4* p = a.W + ((size_t)nxt * a.ksteps + s0) * 64 + lane;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            acc = mfma_16x16x32(ah[s], wb[s], acc);
            accl = mfma_16x16x32(al[s], wb[s], accl);
            if (more) wb[s] = load_stream(p + (size_t)s * 64);
        }
        if (threadIdx.x == 0) next_s[(it + 1) & 1] = nxt < T ? min(G + (int)grab, T) : T;
        const int parity = it & 1;
        red[parity][wave][lane] = acc + accl;
        __syncthreads();
        cur = nxt;
        if (wave / FIN == it % groups) {
            const float* rp = (const float*)&red[parity][0][lane];
            const int i = wave % FIN, m = 4 * g + i;
            float v = rp[i];
#pragma unroll
            for (int w = 1; w < NW; ++w) v += rp[w * 256 + i];   // fixed order over the K-slices
            float2 tl;
            const unsigned long long key = epi_lmhead(a, v * inv_s[m], m, t, lane, &tl);
            if (r == 0) {
                key_s[wave][m] = umax64(key_s[wave][m], key);
                if (a.part_lse) lse_s[wave][m] = lse_merge(lse_s[wave][m], tl);
            }
        }
    }

    NLD_TS(TL_LM, 2);
    // one argmax key per row for this workgroup
    __syncthreads();
    if ((int)threadIdx.x < a.M && threadIdx.x < 16) {
        unsigned long long best = 0ull;
        for (int w = 0; w < NW; ++w) best = umax64(best, key_s[w][threadIdx.x]);
        a.part_keys[(size_t)threadIdx.x * a.n_keys + blockIdx.x] = best;
        if (a.part_lse) {
            float2 st = float2{-INFINITY, 0.f};
            for (int w = 0; w < NW; ++w) st = lse_merge(st, lse_s[w][threadIdx.x]);
            a.part_lse[(size_t)threadIdx.x * a.n_parts + blockIdx.x] = st;
        }
    }
}

constexpr int NORM_NW = 8, NORM_KS = 16;
int gemm_norm_ksteps() { return NORM_NW * NORM_KS; }

hipError_t launch_gemm_norm(int grid, const GemmArgs& a, hipStream_t s) {
    if (a.M > 16 || a.ksteps != NORM_NW * NORM_KS) return hipErrorInvalidValue;
    launch(gemm_norm_kernel<NORM_NW, NORM_KS>, dim3(grid), dim3(NORM_NW * 64), s, a);
    return hipGetLastError();
}

// =====================================================================================
// Streamed GEMM: the O projection of up to 16 rows.  A workgroup takes one column tile; its NW wavefronts
// split the reduction, each streaming its slice of the weights and of the split activations with one batch
// in flight ahead of the MFMAs (two per weight operand).  No slices meet and rows past M are not read: in the middle of a
// pass 8.6 us at 1 and 8 rows of the 8B shapes against 11.9 us for the panel GEMM, 10.8 against 12.3 at 16.  XK: the reduction
// continues over a second source (the LoRA up-projection): 11.1 us with rank 128 at 16 rows of the 8B shapes.  The
// zeros past the ends are written as values: a conditional between a named zero quad and a loaded one chooses an
// address, and the quad then lives in private memory (16.9 us).
// =====================================================================================
// Operand and weight registers of one batch: U k-steps of CT column tiles.
template <int CT, int U>
struct Batch {
    uint4 w[U][CT];
    uint4 x[U];
    uint4 xl[U];
};

template <int NW, bool XK>
__global__ void __launch_bounds__(NW * 64) gemm_stream_kernel(GemmArgs a) {
    constexpr int U = NW > 8 ? 4 : 8;   // 16 wavefronts (at most 128 registers each): half the batch
    typedef Batch<1, U> B;
    __shared__ f32x4_t red[NW][64];
    NLD_TS(TL_O, 0);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int t = blockIdx.x;
    const int per = (a.ksteps + NW - 1) / NW;
    const int s_begin = min(a.ksteps, wave * per), s_end = min(a.ksteps, s_begin + per);
    const uint4* wp = a.W + (size_t)t * a.ksteps * 64 + lane;
    const uint16_t* ap = a.A + (size_t)lane * 8;
    const bool aok = r < a.M;

    // XK: the second source's k-steps (W2 against A2) go one to a wavefront (wavefront w takes step
    // w, then w + NW).  They are loaded before the main stream and multiplied after it, so the
    // main loop is the same as without them.
    constexpr int XS = XK ? 2 : 1;   // second-source k-steps held per wavefront (at most 2 * NW in all)
    uint4 xw[XS], xa[XS], xal[XS];
    if constexpr (XK) {
#pragma unroll
        for (int i = 0; i < XS; ++i) {
            const int s2 = wave + i * NW;
            const bool in = s2 < a.ksteps2;
            const uint16_t* ap2 = a.A2 + (size_t)s2 * 1024 + (size_t)lane * 8;
            xw[i] = in ? a.W2[((size_t)t * a.ksteps2 + s2) * 64 + lane] : uint4{0u, 0u, 0u, 0u};
            xa[i] = in && aok ? *(const uint4*)ap2 : uint4{0u, 0u, 0u, 0u};
            xal[i] = in && aok ? *(const uint4*)(ap2 + SPLIT_LO) : uint4{0u, 0u, 0u, 0u};
        }
    }

    // Epilogue: wavefront i < 4 takes rows 4g + i; its residual value and next gain are fetched up front so
    // that the epilogue waits on no load.
    const int m = 4 * g + wave;
    float xres = 0.f, gn = 0.f;
    if (wave < 4) {
        gn = bf16_to_f32(a.gain_next[t * 16 + r]);
        if (m < a.M) xres = a.x[(size_t)m * a.n_tiles * 16 + t * 16 + r];
    }

    f32x4_t acc = {0.f, 0.f, 0.f, 0.f}, accl = {0.f, 0.f, 0.f, 0.f};
    auto load = [&](int s, B& buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int ss = s + u;
            const bool in = ss < s_end, ok = in && aok && ss * 32 + 8 * g < a.K;
            buf.w[u][0] = in ? wp[(size_t)ss * 64] : uint4{0u, 0u, 0u, 0u};
            buf.x[u] = ok ? *(const uint4*)(ap + (size_t)ss * 1024) : uint4{0u, 0u, 0u, 0u};
            buf.xl[u] = ok ? *(const uint4*)(ap + (size_t)ss * 1024 + SPLIT_LO) : uint4{0u, 0u, 0u, 0u};
        }
    };
    auto compute = [&](const B& buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc = mfma_16x16x32(buf.x[u], buf.w[u][0], acc);
            accl = mfma_16x16x32(buf.xl[u], buf.w[u][0], accl);
        }
    };
    B b0, b1;
    load(s_begin, b0);
    for (int s = s_begin; s < s_end; s += 2 * U) {
        load(s + U, b1);
        compute(b0);
        load(s + 2 * U, b0);
        compute(b1);
    }

    NLD_TS(TL_O, 1);   // main loop done
    if constexpr (XK) {
#pragma unroll
        for (int i = 0; i < XS; ++i) {
            acc = mfma_16x16x32(xa[i], xw[i], acc);
            accl = mfma_16x16x32(xal[i], xw[i], accl);
        }
    }
    red[wave][lane] = acc + accl;
    __syncthreads();
    if (wave < 4) {
        const float* rp = (const float*)&red[0][lane];
        float v = rp[wave];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += rp[w * 256 + wave];   // fixed order over the K-slices
        epi_resid(a, v, m, t, lane, xres, gn);
    }
#ifdef NLD_TIMELINE
    __syncthreads();
#endif
    NLD_TS(TL_O, 2);
}

hipError_t launch_gemm_stream(int nw, const GemmArgs& a, hipStream_t s) {
    if (a.M > 16 || (a.W2 && a.ksteps2 > 16)) return hipErrorInvalidValue;
    const dim3 grid(a.n_tiles);
    if (a.W2) launch(gemm_stream_kernel<8, true>, grid, dim3(512), s, a);   // its k-steps need these registers
    else if (nw == 16) launch(gemm_stream_kernel<16, false>, grid, dim3(1024), s, a);
    else if (nw == 8) launch(gemm_stream_kernel<8, false>, grid, dim3(512), s, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// =====================================================================================
// Split-K GEMM: the down projection of up to 8 rows, where two K slices per column group fit the CUs (rows past M are
// not read; both sides' times stand at the rule, plan_splitk).
// Workgroup (column group cg,
// K slice ks) multiplies its slice of the operand against CT column tiles, so the
// operand is read once per CT tiles and K slice instead of once per tile (the split
// operand is twice as large as the weights it multiplies in these projections).  The
// NW wavefronts cut the slice further and meet in LDS.  With ksplit > 1 the workgroup's
// partial [16 rows][16*CT columns] goes to the workspace with agent-scope stores
// (written through to memory, so that every XCD sees them); once every lane's stores
// are acknowledged, one atomic on the group's counter counts the workgroup in.  The
// workgroup that arrives last reads the other partials with agent-scope loads (which
// do not hit stale lines of its own L2), adds the ksplit partials in slice order (the
// sum does not depend on which workgroup is last), sets the counter back to zero for
// the next launch and runs the residual epilogue.  No workgroup ever waits for
// another: there is no spin and no cache-wide fence.
// =====================================================================================
template <int CT, int NW>
__global__ void __launch_bounds__(NW * 64) gemm_splitk_kernel(GemmArgs a, float* part, unsigned* ctr, int ksplit) {
    constexpr int U = CT <= 3 ? 4 : 2;   // k-steps per batch (the registers of 2 + CT operand quads each)
    typedef Batch<CT, U> B;
    static_assert(CT <= NW, "a wavefront finishes at most one tile");
    __shared__ f32x4_t red[NW][CT][64];
    __shared__ int last_s;
    // timeline class: a reduction longer than the output is the down projection's
    const int TLC = a.K > a.n_tiles * 16 ? TL_DOWN : TL_O;
    (void)TLC;
    NLD_TS(TLC, 0);

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int cg = blockIdx.x, ks = blockIdx.y;
    const int t0 = cg * CT;
    const int N = a.n_tiles * 16;

    // the workgroup's k-steps [kb, ke), then the wavefront's share [s_begin, s_end)
    const int per_wg = (a.ksteps + ksplit - 1) / ksplit;
    const int kb = min(a.ksteps, ks * per_wg), ke = min(a.ksteps, kb + per_wg);
    const int per = (ke - kb + NW - 1) / NW;
    const int s_begin = min(ke, kb + wave * per);
    const int s_end = min(ke, s_begin + per);

    // epilogue inputs of this wavefront's tile (wavefronts past CT have none), fetched up front: residual rows
    // 4g + i of the tile and the next RMSNorm gain of column r
    const int t = t0 + wave;
    const bool mine = wave < CT && t < a.n_tiles;
    float xres[4] = {0.f, 0.f, 0.f, 0.f}, gn = 0.f;
    if (mine) {
        gn = bf16_to_f32(a.gain_next[t * 16 + r]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * g + i < a.M) xres[i] = a.x[(size_t)(4 * g + i) * N + t * 16 + r];
    }

    const uint4* wp[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) wp[ct] = a.W + (size_t)min(t0 + ct, a.n_tiles - 1) * a.ksteps * 64 + lane;
    const bool aok = r < a.M;
    const uint16_t* ap = a.A + (size_t)lane * 8;

    f32x4_t acc[CT], accl[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        acc[ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        accl[ct] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }

    const uint4 zero4 = {0u, 0u, 0u, 0u};
    auto load = [&](int s, B& buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int ss = s + u;
            const bool in = ss < s_end, ok = in && aok && ss * 32 + 8 * g < a.K;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) buf.w[u][ct] = in ? wp[ct][(size_t)ss * 64] : zero4;
            buf.x[u] = ok ? *(const uint4*)(ap + (size_t)ss * 1024) : zero4;
            buf.xl[u] = ok ? *(const uint4*)(ap + (size_t)ss * 1024 + SPLIT_LO) : zero4;
        }
    };
    auto compute = [&](const B& buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                acc[ct] = mfma_16x16x32(buf.x[u], buf.w[u][ct], acc[ct]);
                accl[ct] = mfma_16x16x32(buf.xl[u], buf.w[u][ct], accl[ct]);
            }
    };

    B b0, b1;
    load(s_begin, b0);
    for (int s = s_begin; s < s_end; s += 2 * U) {
        load(s + U, b1);
        compute(b0);
        load(s + 2 * U, b0);
        compute(b1);
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) red[wave][ct][lane] = acc[ct] + accl[ct];
    __syncthreads();
    NLD_TS(TLC, 1);   // main loop done

    // the workgroup's partial of the wavefront's tile (fixed order over the wavefronts), kept in registers and,
    // with ksplit > 1, stored for the last workgroup
    typedef unsigned long long u64;
    f32x4_t v = {0.f, 0.f, 0.f, 0.f};
    if (wave < CT) {
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red[w][wave][lane];
    }
    if (ksplit > 1) {
        auto at = [&](int sl) { return (u64*)(part + ((((size_t)cg * ksplit + sl) * CT + wave) * 64 + lane) * 4); };
        if (wave < CT) {
            u64* pp = at(ks);
            __hip_atomic_store(pp, __builtin_bit_cast(u64, f32x2_t{v[0], v[1]}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(pp + 1, __builtin_bit_cast(u64, f32x2_t{v[2], v[3]}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // every lane's stores are acknowledged before the workgroup counts itself in
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __syncthreads();
        if (threadIdx.x == 0)
            last_s = __hip_atomic_fetch_add(ctr + cg, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(ksplit - 1);
        __syncthreads();
        NLD_TS(TLC, 2);   // partial counted in
        if (!last_s) return;
        if (threadIdx.x == 0) __hip_atomic_exchange(ctr + cg, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (wave < CT) {
            f32x4_t sum = {0.f, 0.f, 0.f, 0.f};
            for (int sl = 0; sl < ksplit; ++sl) {
                if (sl == ks) {
                    sum += v;
                    continue;
                }
                const u64* qq = at(sl);
                const f32x2_t lo = __builtin_bit_cast(f32x2_t, __hip_atomic_load(qq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                const f32x2_t hi = __builtin_bit_cast(f32x2_t, __hip_atomic_load(qq + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                sum += f32x4_t{lo[0], lo[1], hi[0], hi[1]};
            }
            v = sum;
        }
    }
    if (!mine) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) epi_resid(a, v[i], 4 * g + i, t, lane, xres[i], gn);
}

hipError_t launch_gemm_splitk(int ct, int ksplit, const GemmArgs& a, float* part, unsigned* ctr, hipStream_t s) {
    if (a.M > 16 || a.W2 || ct < 2 || ct > 4 || ksplit < 1 || ksplit > SPLITK_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((a.n_tiles + ct - 1) / ct), (unsigned)ksplit), blk(512);
    if (ct == 4) launch(gemm_splitk_kernel<4, 8>, grid, blk, s, a, part, ctr, ksplit);
    else if (ct == 3) launch(gemm_splitk_kernel<3, 8>, grid, blk, s, a, part, ctr, ksplit);
    else launch(gemm_splitk_kernel<2, 8>, grid, blk, s, a, part, ctr, ksplit);
    return hipGetLastError();
}

// =====================================================================================
// Panel GEMM: every projection, except where the three kernels above are faster at up to 16 rows (the LM
// head of a long vocabulary, O, and down up to 8 rows).  A workgroup of 8 wavefronts
// computes 16*RT rows x 16*WC*CT columns over one K slice: WC wavefronts side by side, each with
// CT column tiles against all RT row tiles, times WK = 8 / WC wavefront groups that take the
// k-steps of a stage in turn and meet in LDS at the end.
//
// What bounds it and why this split.  A CU takes in about 25 GB/s of weights while all 256 stream
// from HBM and about 95 GB/s from L2, and the two add up: the time is close to weights / 6.3 TB/s +
// operand bytes per CU / 95 GB/s.  So the split operand (2 KiB per row tile and k-step, twice a
// weight tile) goes through LDS once per workgroup and is shared by wavefronts that lie side by side
// in columns; each weight block has one reader and goes straight to that wavefront's registers.  A
// wavefront's RT x CT tile also sets the LDS rate: it reads 2 RT KiB per k-step for RT*CT pairs of
// MFMAs, so CT = 3 at RT = 8 keeps the matrix cores ahead of LDS (8 x 2 just matches it).  Two
// wavefronts per SIMD cover each other's barrier and LDS latency (four wavefronts of 8 x 6 tiles:
// 176 us against 154 for gate/up at 512 rows).
//
// Stages are KB k-steps.  Stage s is multiplied from LDS slot s & 1 and weight registers s & 1;
// a weight block's register is refilled with its stage s + 2 as soon as it has been multiplied, and
// the operand of stage s + 1 (loaded two stages before) is stored to the other slot while stage s is
// multiplied.  The weights are the MFMA's A operand, so a lane ends up with four neighbouring columns
// of one row (lane 16g + r: row r, columns 4g .. 4g+3) and every epilogue stores 8 or 16 bytes.
//
// K slices (grid) meet like the split-K GEMM's: agent-scope partials, one counter per tile group,
// the last arriver adds the slices in slice order and runs the epilogue.  K steps that do not fill a
// stage, and the second source (LoRA), are multiplied after the loop, straight from global memory.
// =====================================================================================
// A thread's share of the sums of squares of a workgroup's ROWS rows: row threadIdx.x / TPR, partial sums
// threadIdx.x % TPR, + TPR, ...  Requested before the main loop's first loads, added up after them, so that
// the round trip hides behind theirs (row after row in front of the loop took 4 to 9 us per launch).
template <int ROWS, int NT>
struct RowSums {
    static constexpr int TPR = NT / ROWS, U = 16;
    float t[U];
    __device__ __forceinline__ void load(const GemmArgs& a, int m0) {
        const float* ps = a.part_ss + (size_t)(m0 + threadIdx.x / TPR) * a.n_ss;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = (int)threadIdx.x % TPR + u * TPR;
            t[u] = p < a.n_ss ? ps[p] : 0.f;
        }
    }
    // 1/rms per row into inv_s; rows past M get 0
    __device__ __forceinline__ void finish(const GemmArgs& a, int m0, float* inv_s) {
        const int row = threadIdx.x / TPR;
        float s = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) s += t[u];
        const float* ps = a.part_ss + (size_t)(m0 + row) * a.n_ss;
        for (int p = (int)threadIdx.x % TPR + U * TPR; p < a.n_ss; p += TPR) s += ps[p];
#pragma unroll
        for (int off = 1; off < TPR; off <<= 1) s += __shfl_xor(s, off);
        if (threadIdx.x % TPR == 0) inv_s[row] = m0 + row < a.M ? 1.0f / sqrtf(s / (float)a.K + a.eps) : 0.f;
    }
};

// ---- epilogues of four neighbouring columns n = 16t + 4g + i of row m (lane 16g + r: row r of the row tile)
__device__ __forceinline__ void store_split4(uint16_t* p, size_t hi_index, const float* v, uint32_t plain) {
    uint32_t h[2], l[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        h[q] = pack_bf16x2(v[2 * q], v[2 * q + 1]);
        l[q] = plain ? 0u : pack_bf16x2(v[2 * q] - bf16_to_f32(h[q] & 0xFFFFu), v[2 * q + 1] - bf16_to_f32(h[q] >> 16));
    }
    *(uint2*)(p + hi_index) = uint2{h[0], h[1]};
    *(uint2*)(p + hi_index + SPLIT_LO) = uint2{l[0], l[1]};
}

// One column tile of the QKV projection, decoded once for all its row tiles (t is uniform).
struct QkvTile {
    int kind, dim, head_q, row_q, kvh;   // kind 0 q, 1 k, 2 v; q: KV head and first block row of the head's rows
    size_t dpart;                        // q: the head dimensions' share of q_index
    __device__ __forceinline__ void decode(const GemmArgs& a, int t, int g) {
        const int D = a.head_dim, tph = D / 16, hh = t / tph, u = t % tph, nq = a.n_q_heads, nkv = a.n_kv_heads;
        kind = hh < nq ? 0 : (hh < nq + nkv ? 1 : 2);
        dim = 8 * u + 4 * (g & 1) + (g < 2 ? 0 : D / 2);   // lanes g and g ^ 2 hold RoPE partners
        const int G = nq / nkv;
        head_q = hh / G;
        row_q = (hh % G) * a.k_blk;
        kvh = hh - nq - (kind == 2 ? nkv : 0);
        dpart = (size_t)(dim >> 5) * 1024 + (((dim & 31) >> 3) << 7) + (dim & 7);
    }
};

// Four columns of row m (sequence b, block row jb, absolute position pos); c0, c1: the (cos, sin) pairs of
// their rotary frequencies.
__device__ __forceinline__ void epi4_qkv(const GemmArgs& a, const QkvTile& tl, f32x4_t y, int m, int b, int jb, int pos,
                                         int g, float4 c0, float4 c1) {
    const int D = a.head_dim, nkv = a.n_kv_heads;
    float out[4] = {y[0], y[1], y[2], y[3]};
    if (tl.kind < 2) {
        const float co[4] = {c0.x, c0.z, c1.x, c1.z}, si[4] = {c0.y, c0.w, c1.y, c1.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float partner = __shfl_xor(y[i], 32);
            out[i] = g < 2 ? (y[i] * co[i] - partner * si[i]) : (y[i] * co[i] + partner * si[i]);
        }
    }
    if (m >= a.M) return;
    if (tl.kind == 0) {   // q_index(b * nkv + head_q, row_q + jb, dim, ...)
        const int row = tl.row_q + jb;
        const size_t at = (size_t)((b * nkv + tl.head_q) * a.q_row_tiles + (row >> 4)) * ((D >> 5) * 1024) + (row & 15) * 8;
        store_split4(a.q_out, at + tl.dpart, out, a.plain & SITE_Q);
        return;
    }
    const size_t unit = (size_t)b * nkv + tl.kvh;
    const int dim = tl.dim;
    const bool cache = a.write_cache && !(a.quad_k > 0 && jb >= a.quad_k);   // quadratic layout: chain rows only
    if (cache && pos >= a.max_len) atomicOr(a.status, DEV_CAPACITY);
    const bool wr = cache && pos < a.max_len;
    uint32_t h[2], l[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        h[q] = pack_bf16x2(out[2 * q], out[2 * q + 1]);
        l[q] = (a.plain & SITE_KV)
                   ? 0u
                   : pack_bf16x2(out[2 * q] - bf16_to_f32(h[q] & 0xFFFFu), out[2 * q + 1] - bf16_to_f32(h[q] >> 16));
    }
    if (tl.kind == 1) {
        *(uint2*)(a.blk_k + (unit * 2 * 64 + jb) * D + dim) = uint2{h[0], h[1]};
        *(uint2*)(a.blk_k + ((unit * 2 + 1) * 64 + jb) * D + dim) = uint2{l[0], l[1]};
        if (wr) *(uint2*)(a.kc + (unit * a.max_len + pos) * D + dim) = uint2{h[0], h[1]};
        return;
    }
    uint16_t* bv = a.blk_v + (unit * 2 * D + dim) * 64 + jb;   // values are stored transposed
    uint16_t* cv = a.vc + ((unit * (a.max_len / 64) + pos / 64) * D + dim) * 64 + (pos & 63);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint16_t hb = (uint16_t)(h[i >> 1] >> (16 * (i & 1))), lb = (uint16_t)(l[i >> 1] >> (16 * (i & 1)));
        bv[i * 64] = hb;
        bv[(size_t)D * 64 + i * 64] = lb;
        if (wr) cv[i * 64] = hb;
    }
}

// y * sigmoid(y).  The library's exponential and the divide, which are right over the whole range (an overflowing
// exp(-y) gives -0) and within 2.8 ulp.  A hardware exp2 with its argument's remainder and a reciprocal are within
// 3.7 ulp and gave NaN where the remainder meets an infinite exp2 (gates from -88.73 to -104); they saved 6 of 902 us a
// pass at 120 rows of the 8B shapes, four layers.
__device__ __forceinline__ float silu(float y) { return y / (1.0f + expf(-y)); }

// rotation of the 16 lanes of a row by N (a register move, where a shuffle goes through LDS)
template <int N>
__device__ __forceinline__ uint32_t row_ror(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x120 | N, 0xF, 0xF, true);
}
template <int N>
__device__ __forceinline__ float row_ror(float v) { return __uint_as_float(row_ror<N>(__float_as_uint(v))); }

// Lanes g < 2 hold four gate columns, lanes g ^ 2 the matching up columns; each lane of a pair finishes two
// of the four columns.
__device__ __forceinline__ void epi4_swiglu(const GemmArgs& a, f32x4_t y, int m, int t, int g) {
    const bool lowg = g < 2;
    const float r0 = __shfl_xor(lowg ? y[2] : y[0], 32), r1 = __shfl_xor(lowg ? y[3] : y[1], 32);
    const float a0 = silu(lowg ? y[0] : r0) * (lowg ? r0 : y[2]), a1 = silu(lowg ? y[1] : r1) * (lowg ? r1 : y[3]);
    const int col = 8 * t + 4 * (g & 1) + (lowg ? 0 : 2);
    if (m < a.M && col < a.ffn) {   // ffn is a multiple of 8: the tile's columns are in or out together
        const uint32_t h = pack_bf16x2(a0, a1);
        const uint32_t l = (a.plain & SITE_ACT) ? 0u : pack_bf16x2(a0 - bf16_to_f32(h & 0xFFFFu), a1 - bf16_to_f32(h >> 16));
        uint16_t* p = a.act + split_index(m, col, (a.ffn + 31) / 32);
        *(uint32_t*)p = h;
        *(uint32_t*)(p + SPLIT_LO) = l;
    }
}

// returns the sum of squares of the four new residual values
__device__ __forceinline__ float epi4_resid(const GemmArgs& a, f32x4_t v, int m, int t, int g, float4 xr, uint2 gn) {
    if (m >= a.M) return 0.f;
    const int N = a.n_tiles * 16, n = t * 16 + 4 * g;
    const float xn[4] = {xr.x + v[0], xr.y + v[1], xr.z + v[2], xr.w + v[3]};
    *(float4*)(a.x + (size_t)m * N + n) = float4{xn[0], xn[1], xn[2], xn[3]};
    const float xg[4] = {xn[0] * bf16_to_f32(gn.x & 0xFFFFu), xn[1] * bf16_to_f32(gn.x >> 16),
                         xn[2] * bf16_to_f32(gn.y & 0xFFFFu), xn[3] * bf16_to_f32(gn.y >> 16)};
    store_split4(a.xg_out, split_index(m, n, N / 32), xg, a.plain & (SITE_NORM | SITE_FINAL));
    return (xn[0] * xn[0] + xn[1] * xn[1]) + (xn[2] * xn[2] + xn[3] * xn[3]);
}

// 16 bytes per lane at agent scope: what an agent-scope atomic store or load of 8 bytes compiles to (the
// sc1 bit: through this XCD's L2, to and from where every XCD sees it), at twice the width.  `p` is the
// lane's address; the buffer descriptor takes the first lane's as its base.
constexpr int CPOL_AGENT = 16;   // sc1
__device__ __forceinline__ __amdgpu_buffer_rsrc_t agent_rsrc(const void* p, uint32_t* off) {
    const uint64_t at = (uint64_t)p;
    const uint64_t base = (uint64_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32)) << 32 |
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at);
    *off = (uint32_t)(at - base);
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7FFFFFFF, 0x00027000);
}
__device__ __forceinline__ void store_agent(f32x4_t* p, f32x4_t v) {
    typedef uint32_t u32x4_b __attribute__((ext_vector_type(4)));
    uint32_t off;
    const __amdgpu_buffer_rsrc_t rs = agent_rsrc(p, &off);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_b, v), rs, off, 0, CPOL_AGENT);
}
__device__ __forceinline__ f32x4_t load_agent(const f32x4_t* p) {
    uint32_t off;
    const __amdgpu_buffer_rsrc_t rs = agent_rsrc(p, &off);
    return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, CPOL_AGENT));
}

template <int RT, int WC, int CT, int KB, int EPI>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
gemm_panel_kernel(GemmArgs a, int R, int C, int ksplit, float* part, unsigned* ctr) {
    constexpr int NW = 8, WK = NW / WC, KW = KB / WK, NT = NW * 64;
    constexpr int BLOCKS = RT * KB * 2;       // 1 KiB operand blocks per stage
    constexpr int APW = BLOCKS / NW;          // of them per wavefront
    constexpr int NTL = RT * CT;              // output tiles per wavefront
    constexpr bool NORMED = EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_LMHEAD;
    static_assert(WC * WK == NW && KW * WK == KB && BLOCKS % NW == 0, "whole shares per wavefront");
    constexpr int RED = WK > 1 ? NW * NTL : 0;   // 1 KiB blocks the k groups meet in
    // Epilogue: a wavefront's tiles pass through LDS in PASSES runs of row tiles, so that the code of one row
    // tile is a loop body.  Unrolled over the accumulators it ran once, straight from a cold instruction
    // cache: 15-40 us per launch at 128 x 384.
    constexpr int PASSES = NTL > 16 ? 4 : (NTL > 12 ? 2 : 1), RPP = RT / PASSES, STG = NW * RPP * CT;
    constexpr int ROPE = EPI == EPI_QKV ? (RT * 16 * 33 + 63) / 64 : 0;   // the rows' RoPE pairs (epilogue)
    constexpr int LDS0 = 2 * BLOCKS > RED ? 2 * BLOCKS : RED, LDS1 = STG + ROPE, LDSB = LDS0 > LDS1 ? LDS0 : LDS1;
    __shared__ uint4 lds[LDSB * 64];
    __shared__ float inv_s[RT * 16];
    __shared__ int pos_s[RT * 16];
    __shared__ int seq_s[RT * 16];   // sequence << 6 | block row (at most 64 of them)
    __shared__ float ss_s[NW][RT * 16];
    __shared__ unsigned long long key_s[NW][RT * 16];
    __shared__ float2 lse_s[NW][RT * 16];
    __shared__ int last_s;
    constexpr int TLC = EPI == EPI_QKV ? TL_QKV : (EPI == EPI_SWIGLU ? TL_GATE_UP : (EPI == EPI_LMHEAD ? TL_LM : TL_DOWN));
    (void)TLC;
    NLD_TS(TLC, 0);

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int wc = wave % WC, wk = wave / WC;
    // Workgroup b runs on XCD b % 8.  Logical id: row group fastest, then column group, then K slice,
    // consecutive ids on one XCD, so that the row groups of a column group find its weights, and the
    // column groups of a slice their operand, in that XCD's L2.
    const int per = gridDim.x / 8;
    const int id = (int)blockIdx.x < per * 8 ? (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
    const int rg = id % R, cg = (id / R) % C, ksl = id / (R * C);
    const int m0 = rg * RT * 16;

    RowSums<RT * 16, NT> sums;
    if constexpr (NORMED) sums.load(a, m0);
    // whole stages of full k-steps, cut into ksplit near-equal runs; the rest is the tail
    const int full = a.K / 32;
    const int nst_all = full / KB;
    const int st0 = ksl * nst_all / ksplit, nst = (ksl + 1) * nst_all / ksplit - st0;

    // The lo products have accumulators of their own where the registers allow it (at most 12 tiles), so that they
    // do not round at the hi sum's size; elsewhere they share the hi products'.
    constexpr bool TWO = RT == 1 || (RT == 2 && (EPI == EPI_QKV || EPI == EPI_RESID)) || EPI == EPI_SPLIT;
    f32x4_t acc[RT][CT], accl[TWO ? RT : 1][TWO ? CT : 1];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < CT; ++j) {
            acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if constexpr (TWO) accl[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }

    // LM head: rows 4g+i of column r instead, so that a logits store is 64 contiguous bytes per row
    auto mm = [](uint4 w, uint4 x, f32x4_t c) __attribute__((always_inline)) {
        return EPI == EPI_LMHEAD ? mfma_16x16x32(x, w, c) : mfma_16x16x32(w, x, c);
    };
    auto mm_lo = [&](uint4 w, uint4 x, int i, int c) __attribute__((always_inline)) {
        if constexpr (TWO) accl[i][c] = mm(w, x, accl[i][c]);
        else acc[i][c] = mm(w, x, acc[i][c]);
    };

    // this wavefront's operand blocks of a stage: blocks wave*APW .. +APW of [row tile][k-step][hi, lo]
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    const u32x4_t* ap[APW];
#pragma unroll
    for (int q = 0; q < APW; ++q) {
        const int ch = wave * APW + q, rt = ch / (KB * 2), in = ch % (KB * 2);
        ap[q] = (const u32x4_t*)a.A + ((size_t)((m0 / 16 + rt) * a.ksteps + st0 * KB) * 2 + in) * 64;
    }
    const uint4* wp[CT];   // column tiles past the end are read clamped and their outputs dropped
#pragma unroll
    for (int c = 0; c < CT; ++c) {
        const int t = min((cg * WC + wc) * CT + c, a.n_tiles - 1);
        wp[c] = a.W + ((size_t)t * a.ksteps + st0 * KB + wk * KW) * 64;
    }

    if (nst > 0) {
        u32x4_t ar[2][APW];
        uint4 wr[2][KW][CT];
#define NLD_PANEL_LDA(st, set)                                                      \
    {                                                                               \
        const size_t so_ = (size_t)min((st), nst - 1) * KB * 128;                   \
        _Pragma("unroll") for (int q = 0; q < APW; ++q) ar[set][q] = ap[q][so_ + lane]; \
    }
#define NLD_PANEL_LDW(st, set, kk)                                                  \
    {                                                                               \
        const size_t so_ = (size_t)(min((st), nst - 1) * KB + (kk)) * 64;           \
        _Pragma("unroll") for (int c = 0; c < CT; ++c) wr[set][kk][c] = load_stream(wp[c] + so_ + lane); \
    }
#define NLD_PANEL_STA(set, slot)                                                    \
    _Pragma("unroll") for (int q = 0; q < APW; ++q)                                 \
        *(u32x4_t*)&lds[((slot) * BLOCKS + wave * APW + q) * 64 + lane] = ar[set][q];
        NLD_PANEL_LDA(0, 0);
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int kk = 0; kk < KW; ++kk) NLD_PANEL_LDW(p, p, kk);
        NLD_PANEL_LDA(1, 1);
        if constexpr (NORMED) sums.finish(a, m0, inv_s);
        NLD_PANEL_STA(0, 0);
        NLD_PANEL_LDA(2, 0);
        __syncthreads();
        NLD_TS(TLC, 3);   // first stage in LDS
        for (int st = 0; st < nst; st += 2) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (st + u >= nst) break;
#pragma unroll
                for (int kk = 0; kk < KW; ++kk) {
#pragma unroll
                    for (int i = 0; i < RT; ++i) {
                        const int bi = (u * BLOCKS + (i * KB + wk * KW + kk) * 2) * 64 + lane;
                        const uint4 ah = lds[bi], al = lds[bi + 64];
#pragma unroll
                        for (int c = 0; c < CT; ++c) acc[i][c] = mm(wr[u][kk][c], ah, acc[i][c]);
#pragma unroll
                        for (int c = 0; c < CT; ++c) mm_lo(wr[u][kk][c], al, i, c);
                    }
                    NLD_PANEL_LDW(st + u + 2, u, kk);
                    if (kk == 0) {
                        NLD_PANEL_STA(u ^ 1, u ^ 1);
                        NLD_PANEL_LDA(st + u + 3, u ^ 1);
                    }
                }
                __syncthreads();
            }
        }
#undef NLD_PANEL_LDA
#undef NLD_PANEL_LDW
#undef NLD_PANEL_STA
    } else if constexpr (NORMED) {
        sums.finish(a, m0, inv_s);
    }

    // the last slice also takes the k-steps that fill no stage (the last may be partial: columns past
    // K meet zeroed operand lanes) and the second source's, the k groups by turns
    if (ksl == ksplit - 1) {
        const int s1 = nst_all * KB, n1 = a.ksteps - s1, n2 = a.W2 ? a.ksteps2 : 0;
        for (int e = wk; e < n1 + n2; e += WK) {
            const bool second = e >= n1;
            const int s = second ? e - n1 : s1 + e, nk = second ? a.ksteps2 : a.ksteps;
            const uint4* wb = second ? a.W2 : a.W;
            const uint16_t* ab = second ? a.A2 : a.A;
            const bool in = second || s * 32 + 8 * g < a.K;
            uint4 w[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) w[c] = wb[((size_t)min((cg * WC + wc) * CT + c, a.n_tiles - 1) * nk + s) * 64 + lane];
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                const uint4* xp = (const uint4*)(ab + (size_t)((m0 / 16 + i) * nk + s) * 1024) + lane;
                const uint4 ah = in ? xp[0] : uint4{0u, 0u, 0u, 0u}, al = in ? xp[64] : uint4{0u, 0u, 0u, 0u};
#pragma unroll
                for (int c = 0; c < CT; ++c) acc[i][c] = mm(w[c], ah, acc[i][c]);
#pragma unroll
                for (int c = 0; c < CT; ++c) mm_lo(w[c], al, i, c);
            }
        }
    }
    NLD_TS(TLC, 1);   // main loop done
    if constexpr (TWO) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < CT; ++j) acc[i][j] += accl[i][j];
    }

    // The k groups meet in LDS (fixed order); group wk keeps tiles wk, wk + WK, ... of its column wavefront.
    if constexpr (WK > 1) {
        f32x4_t* red = (f32x4_t*)lds;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NTL; ++q) red[(wave * NTL + q) * 64 + lane] = acc[q / CT][q % CT];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NTL; ++q) {
            if (q % WK != wk) continue;
            f32x4_t s = red[(wc * NTL + q) * 64 + lane];
#pragma unroll
            for (int w = 1; w < WK; ++w) s += red[((w * WC + wc) * NTL + q) * 64 + lane];
            acc[q / CT][q % CT] = s;
        }
    }

    if (ksplit > 1) {
        // slice partials: one contiguous 1 KiB block per tile
        const int grp = cg * R + rg;
        auto at = [&](int sl) { return (f32x4_t*)part + ((size_t)(grp * ksplit + sl) * WC + wc) * NTL * 64 + lane; };
        f32x4_t* pp = at(ksl);
#pragma unroll
        for (int q = 0; q < NTL; ++q) {
            if (WK > 1 && q % WK != wk) continue;
            store_agent(pp + q * 64, acc[q / CT][q % CT]);
        }
        // every lane's stores are acknowledged before the workgroup counts itself in
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __syncthreads();
        if (threadIdx.x == 0)
            last_s = __hip_atomic_fetch_add(ctr + grp, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(ksplit - 1);
        __syncthreads();
        if (!last_s) return;
        if (threadIdx.x == 0) __hip_atomic_exchange(ctr + grp, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // fixed order over the slices, all of a slice's loads in flight at once (in two halves where the
        // registers of a whole wavefront tile, its sums and its loads do not fit beside each other)
        constexpr int CH = NTL > 16 ? NTL / 2 : NTL;
        static_assert(NTL % CH == 0, "whole chunks");
#pragma unroll
        for (int q0 = 0; q0 < NTL; q0 += CH) {
            f32x4_t sum[CH];
#pragma unroll
            for (int q = 0; q < CH; ++q) sum[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            for (int sl = 0; sl < ksplit; ++sl) {
                if (sl == ksl) {
#pragma unroll
                    for (int q = 0; q < CH; ++q) sum[q] += acc[(q0 + q) / CT][(q0 + q) % CT];
                    continue;
                }
                const f32x4_t* qq = at(sl) + q0 * 64;
                f32x4_t v[CH];
#pragma unroll
                for (int q = 0; q < CH; ++q) {
                    if (WK > 1 && (q0 + q) % WK != wk) continue;
                    v[q] = load_agent(qq + q * 64);
                }
#pragma unroll
                for (int q = 0; q < CH; ++q) {
                    if (WK > 1 && (q0 + q) % WK != wk) continue;
                    sum[q] += v[q];
                }
            }
#pragma unroll
            for (int q = 0; q < CH; ++q) acc[(q0 + q) / CT][(q0 + q) % CT] = sum[q];
        }
    }
    if constexpr (EPI == EPI_QKV) {
        if (threadIdx.x < RT * 16) {
            const int m = min(m0 + (int)threadIdx.x, a.M - 1), b = m / a.k_blk;
            seq_s[threadIdx.x] = b << 6 | (m - b * a.k_blk);
            pos_s[threadIdx.x] = committed_length(a.lengths, b, a.max_len, a.status) + m - b * a.k_blk;
        }
    }
    if constexpr (NORMED) __syncthreads();   // inv_s, pos_s, seq_s
    NLD_TS(TLC, 2);   // slices added

    auto mine = [&](int i, int c) { return WK == 1 || (i * CT + c) % WK == wk; };
    // f(i, tiles) for every row tile i, from the wavefront's own LDS
    auto each_row_tile = [&](auto f) __attribute__((always_inline)) {
        if constexpr (WK > 1) __syncthreads();   // every group has read the others' sums
        f32x4_t* stg = (f32x4_t*)lds + wave * RPP * CT * 64 + lane;
#pragma unroll 1
        for (int ps = 0; ps < PASSES; ++ps) {
#pragma unroll
            for (int p2 = 0; p2 < PASSES; ++p2) {
                if (ps != p2) continue;
#pragma unroll
                for (int q = 0; q < RPP * CT; ++q) stg[q * 64] = acc[p2 * RPP + q / CT][q % CT];
            }
#pragma unroll 1
            for (int i = 0; i < RPP; ++i) {
                f32x4_t v[CT];
#pragma unroll
                for (int c = 0; c < CT; ++c) v[c] = stg[(i * CT + c) * 64];
                f(ps * RPP + i, v);
            }
        }
    };
    if constexpr (EPI == EPI_LMHEAD) {
        const int n0 = (cg * WC + wc) * CT * 16 + r;   // column of the lane in the wavefront's first tile
        bool col[CT], cand[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            col[c] = n0 + 16 * c < a.vocab;
            cand[c] = col[c] && n0 + 16 * c != a.exclude_id;
        }
        each_row_tile([&](int i, const f32x4_t (&v)[CT]) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int ml = 16 * i + 4 * g + e, m = m0 + ml;
                const float inv = inv_s[ml];
                float y[CT];
#pragma unroll
                for (int c = 0; c < CT; ++c) y[c] = v[c][e] * inv;
                if (a.logits && m < a.M) {
                    float* lp = a.logits + (size_t)m * a.vocab + n0;
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                        if (col[c] && mine(i, c)) lp[16 * c] = y[c];
                }
                if (a.ens_logits && m < a.M) {   // quadratic layout: verifier rows (chain row i, mask 1 of group i)
                    const int b = m / a.k_blk, jb = m - b * a.k_blk, qk = a.quad_k;
                    const int ci = jb < qk ? jb : ((jb - qk) % qk == 0 ? qk + (jb - qk) / qk : -1);
                    float* ep = a.ens_logits + ((size_t)b * 2 * qk + ci) * a.vocab + n0;
#pragma unroll
                    for (int c = 0; c < CT; ++c)
                        if (col[c] && ci >= 0 && mine(i, c)) ep[16 * c] = y[c];
                }
                // the order argmax_key gives (-0 as +0), as a signed number; then the lowest column of the largest
                int32_t ord[CT], top = INT32_MIN;
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const int32_t u = __float_as_int(y[c] + 0.0f);
                    const bool take = cand[c] && mine(i, c);
                    ord[c] = take ? (u ^ ((u >> 31) & 0x7FFFFFFF)) : INT32_MIN;
                    top = max(top, ord[c]);
                }
                top = max(top, (int32_t)row_ror<8>((uint32_t)top));
                top = max(top, (int32_t)row_ror<4>((uint32_t)top));
                top = max(top, (int32_t)row_ror<2>((uint32_t)top));
                top = max(top, (int32_t)row_ror<1>((uint32_t)top));
                uint32_t first = 0xFFFFFFFFu;
#pragma unroll
                for (int c = CT - 1; c >= 0; --c) first = ord[c] == top ? (uint32_t)(n0 + 16 * c) : first;
                first = min(first, row_ror<8>(first));
                first = min(first, row_ror<4>(first));
                first = min(first, row_ror<2>(first));
                first = min(first, row_ror<1>(first));
                if (a.part_lse) {
                    float mx = ord[0] != INT32_MIN ? y[0] : -INFINITY;   // NaN, and not the empty set's -inf, where all are NaN
#pragma unroll
                    for (int c = 1; c < CT; ++c) mx = fmaxf(mx, ord[c] != INT32_MIN ? y[c] : -INFINITY);
                    mx = fmaxf(mx, row_ror<8>(mx));
                    mx = fmaxf(mx, row_ror<4>(mx));
                    mx = fmaxf(mx, row_ror<2>(mx));
                    mx = fmaxf(mx, row_ror<1>(mx));
                    float sum = 0.f;
#pragma unroll
                    for (int c = 0; c < CT; ++c) sum += ord[c] != INT32_MIN ? expf(y[c] - mx) : 0.f;
                    sum += row_ror<8>(sum);
                    sum += row_ror<4>(sum);
                    sum += row_ror<2>(sum);
                    sum += row_ror<1>(sum);
                    if (r == 0) lse_s[wave][ml] = float2{mx, sum};
                }
                if (r == 0)   // no column of the row here: the empty key
                    key_s[wave][ml] = top == INT32_MIN ? 0ull
                                                       : ((unsigned long long)((uint32_t)top ^ 0x80000000u) << 32) |
                                                             (unsigned long long)(0xFFFFFFFFu - first);
            }
        });
        __syncthreads();
        if (threadIdx.x < RT * 16) {
            const int m = m0 + threadIdx.x;
            if (m < a.M) {
                unsigned long long best = 0ull;
                float2 st = float2{-INFINITY, 0.f};
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    best = umax64(best, key_s[w][threadIdx.x]);
                    if (a.part_lse) st = lse_merge(st, lse_s[w][threadIdx.x]);
                }
                if (a.n_keys < a.n_parts)
                    __hip_atomic_fetch_max(a.part_keys + (size_t)m * a.n_keys + cg % a.n_keys, best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else a.part_keys[(size_t)m * a.n_keys + cg] = best;
                if (a.part_lse) a.part_lse[(size_t)m * a.n_parts + cg] = st;
            }
        }
    } else {
        // Everything the epilogue reads is read before its first store: a wait for a load also waits for every
        // store issued before it (about 1 us per tile when they alternate: 16-20 us at 128 x 384).  The
        // residual goes to registers, the rows' RoPE pairs to LDS (rows 16 bytes apart in banks).
        float4 xr[EPI == EPI_RESID ? CT : 1][EPI == EPI_RESID ? RT : 1];
        constexpr int RS = 33;   // RoPE row stride in 16-byte pieces (head_dim <= 128)
        if constexpr (EPI == EPI_RESID) {
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    if (WK > 1 && (i * CT + c) % WK != wk) continue;
                    const int m = min(m0 + 16 * i + r, a.M - 1), t = min((cg * WC + wc) * CT + c, a.n_tiles - 1);
                    xr[c][i] = *(const float4*)(a.x + (size_t)m * a.n_tiles * 16 + t * 16 + 4 * g);
                }
        }
        float sq[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i) sq[i] = 0.f;
        const int t0 = (cg * WC + wc) * CT;
        if constexpr (EPI == EPI_QKV) {
            uint4* rope_s = lds + STG * 64;
            const int pr = a.head_dim / 4, rot = a.head_dim / 16;   // 16-byte pieces per row; tiles per head
            const uint4* src = (const uint4*)(a.rope + (size_t)m0 * (a.head_dim / 2));
            __syncthreads();   // the stage buffers are free
            for (int q = threadIdx.x; q < RT * 16 * pr; q += NT) rope_s[(q / pr) * RS + q % pr] = src[q];
            __syncthreads();
            QkvTile tl[CT];
#pragma unroll
            for (int c = 0; c < CT; ++c) tl[c].decode(a, t0 + c, g);
            each_row_tile([&](int i, const f32x4_t (&v)[CT]) __attribute__((always_inline)) {
                const int ml = 16 * i + r, seq = seq_s[ml], pos = pos_s[ml];
                const float inv = inv_s[ml];
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    if (!mine(i, c) || t0 + c >= a.n_tiles) continue;
                    const float4* cs = (const float4*)&rope_s[ml * RS + 4 * ((t0 + c) % rot) + 2 * (g & 1)];
                    epi4_qkv(a, tl[c], v[c] * inv, m0 + ml, seq >> 6, seq & 63, pos, g, cs[0], cs[1]);
                }
            });
        } else if constexpr (EPI == EPI_SWIGLU) {
            each_row_tile([&](int i, const f32x4_t (&v)[CT]) __attribute__((always_inline)) {
                const int ml = 16 * i + r;
                const float inv = inv_s[ml];
#pragma unroll
                for (int c = 0; c < CT; ++c)
                    if (mine(i, c) && t0 + c < a.n_tiles) epi4_swiglu(a, v[c] * inv, m0 + ml, t0 + c, g);
            });
        } else {
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const int t = t0 + c;
                uint2 gn = {0u, 0u};
                if constexpr (EPI == EPI_RESID) gn = *(const uint2*)(a.gain_next + min(t, a.n_tiles - 1) * 16 + 4 * g);
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    if (!mine(i, c) || t >= a.n_tiles) continue;
                    const int m = m0 + 16 * i + r;
                    const f32x4_t v = acc[i][c];
                    if constexpr (EPI == EPI_RESID) sq[i] += epi4_resid(a, v, m, t, g, xr[c][i], gn);
                    else if (m < a.M) {
                        const float sv[4] = {a.out_scale * v[0], a.out_scale * v[1], a.out_scale * v[2], a.out_scale * v[3]};
                        store_split4(a.xg_out, split_index(m, t * 16 + 4 * g, a.n_tiles / 2), sv, 0u);
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            if constexpr (EPI == EPI_RESID) {
                sq[i] += __shfl_xor(sq[i], 16);
                sq[i] += __shfl_xor(sq[i], 32);
                if (g == 0) ss_s[wave][16 * i + r] = sq[i];
            }
        }
        if constexpr (EPI == EPI_RESID) {   // one sum of squares per row and column group
            __syncthreads();
            if (threadIdx.x < RT * 16 && m0 + (int)threadIdx.x < a.M) {
                float s = 0.f;
#pragma unroll
                for (int w = 0; w < NW; ++w) s += ss_s[w][threadIdx.x];
                a.part_ss_out[(size_t)(m0 + threadIdx.x) * C + cg] = s;
            }
        }
    }
#ifdef NLD_TIMELINE
    __syncthreads();
#endif
    NLD_TS(TLC, 4);
}

// The workgroup shapes in use, by row tiles: {row tiles, wavefronts side by side, column tiles per
// wavefront, k-steps per stage}.
static constexpr PanelShape PANEL_SHAPES[] = {
    {2, 8, 1, 2}, {2, 4, 1, 4}, {2, 4, 2, 4}, {2, 4, 3, 2}, {2, 2, 3, 4},
    {4, 8, 1, 2}, {4, 4, 1, 4}, {4, 4, 2, 2}, {4, 4, 3, 2},
    {8, 4, 1, 2}, {8, 8, 1, 2}, {8, 8, 2, 2}, {8, 8, 3, 2},
    {1, 2, 3, 4}, {1, 4, 1, 4}, {1, 8, 1, 4}, {1, 1, 3, 8},
};
int gemm_panel_shapes() { return (int)(sizeof(PANEL_SHAPES) / sizeof(PANEL_SHAPES[0])); }
PanelShape gemm_panel_shape(int i) { return PANEL_SHAPES[i]; }

template <int RT, int WC, int CT, int KB>
static hipError_t launch_panel_epi(int epi, dim3 grid, int R, int C, const GemmArgs& a, int ksplit, float* part,
                                   unsigned* ctr, hipStream_t s) {
    const dim3 blk(512);
    switch (epi) {
        case EPI_QKV: launch(gemm_panel_kernel<RT, WC, CT, KB, EPI_QKV>, grid, blk, s, a, R, C, ksplit, part, ctr); break;
        case EPI_RESID: launch(gemm_panel_kernel<RT, WC, CT, KB, EPI_RESID>, grid, blk, s, a, R, C, ksplit, part, ctr); break;
        case EPI_SWIGLU: launch(gemm_panel_kernel<RT, WC, CT, KB, EPI_SWIGLU>, grid, blk, s, a, R, C, ksplit, part, ctr); break;
        case EPI_LMHEAD: launch(gemm_panel_kernel<RT, WC, CT, KB, EPI_LMHEAD>, grid, blk, s, a, R, C, ksplit, part, ctr); break;
        case EPI_SPLIT:
            if constexpr (WC == 4 && CT == 1) {   // gemm_panel_narrow
                launch(gemm_panel_kernel<RT, WC, CT, KB, EPI_SPLIT>, grid, blk, s, a, R, C, ksplit, part, ctr);
                break;
            }
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_gemm_panel(int epi, int shape, const GemmArgs& a, int ksplit, float* part, unsigned* ctr, hipStream_t s) {
    if (shape < 0 || shape >= gemm_panel_shapes()) return hipErrorInvalidValue;
    const PanelShape p = PANEL_SHAPES[shape];
    // every slice gets at least one stage, slices need their partials and counters
    if (ksplit < 1 || (ksplit > 1 && (ksplit > a.K / 32 / p.kb || !part || !ctr))) return hipErrorInvalidValue;
    if (a.W2 && epi != EPI_RESID) return hipErrorInvalidValue;
    const int R = (a.M + 16 * p.rt - 1) / (16 * p.rt), C = (a.n_tiles + p.wc * p.ct - 1) / (p.wc * p.ct);
    const dim3 grid((unsigned)(R * C * ksplit));
    switch (shape) {
        case 0: return launch_panel_epi<2, 8, 1, 2>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 1: return launch_panel_epi<2, 4, 1, 4>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 2: return launch_panel_epi<2, 4, 2, 4>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 3: return launch_panel_epi<2, 4, 3, 2>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 4: return launch_panel_epi<2, 2, 3, 4>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 5: return launch_panel_epi<4, 8, 1, 2>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 6: return launch_panel_epi<4, 4, 1, 4>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 7: return launch_panel_epi<4, 4, 2, 2>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 8: return launch_panel_epi<4, 4, 3, 2>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 9: return launch_panel_epi<8, 4, 1, 2>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 10: return launch_panel_epi<8, 8, 1, 2>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 11: return launch_panel_epi<8, 8, 2, 2>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 12: return launch_panel_epi<8, 8, 3, 2>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 13: return launch_panel_epi<1, 2, 3, 4>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 14: return launch_panel_epi<1, 4, 1, 4>(epi, grid, R, C, a, ksplit, part, ctr, s);
        case 15: return launch_panel_epi<1, 8, 1, 4>(epi, grid, R, C, a, ksplit, part, ctr, s);
        default: return launch_panel_epi<1, 1, 3, 8>(epi, grid, R, C, a, ksplit, part, ctr, s);
    }
}

// =====================================================================================
// Block-masked GQA attention.  Workgroup = (key split, sequence x KV head, row slice); rows = heads of
// the GQA group x block rows, in tiles of 16.  The committed prefix [0, P) is cut into key splits that
// read the bf16 cache; the block part covers the block's own k keys (causal or bidirectional per the
// mode) from the split K/V the QKV epilogue left in the workspace, so this pass sees its own keys and
// values at about 16 significant bits while the cache keeps bf16.  With one sequence the block part is a
// workgroup of its own; in a batch the last split of a unit takes it along.
//
// Keys stream through LDS in stages of 64 (K rows and the transposed V tile, XOR-swizzled for
// conflict-free operand reads).  The stages go from global memory straight to LDS (global_load_lds, the
// swizzle on the global side), so no register holds keys on their way: with NS = 2 slots the kernel fits
// 128 registers and two workgroups share a CU, one loading while the other computes; a batch has work for
// both.  One sequence has at most one workgroup per CU and takes NS = 4, three stages ahead.  (Staged through
// registers the kernel took 224 registers, one workgroup per CU: ten round trips of latency in a row.)
//
// KH = 2 (up to four row tiles): two wavefronts per row tile, each with half of a stage's keys; KH = 1: one.
// S^T = K Q^T on MFMA puts one query row per lane column, so a row's softmax statistics live in lanes r, r+16,
// r+32, r+48 and P^T is already the B operand of O^T = V^T P^T.  Queries and P are split operands.  Online
// softmax in base 2, fp32; every workgroup writes one partial (max, sum, unnormalised output) per row for the
// merge.
// =====================================================================================
template <int D>
struct AttnCfg {
    static constexpr int KCH = D / 8;                    // 16-byte chunks per K row
    static constexpr int KCHUNKS = 64 * KCH;             // K tile chunks per stage
    static constexpr int VCHUNKS = D * 8;                // V tile chunks per stage (D rows x 64 keys)
    static constexpr int CHUNKS = KCHUNKS + VCHUNKS;
    static constexpr int BLOCKS = CHUNKS / 64;           // 1 KiB blocks per stage
};

// XOR swizzles (chunk index within a row): make the 16 rows read by one MFMA
// operand load hit 16 distinct bank groups.
template <int D>
__device__ __forceinline__ int kswz(int row) {
    if constexpr (D == 128) return (row & 3) | ((row >> 1) & 12);
    else return ((row >> 1) & 1) | ((row >> 2) & 6);
}
__device__ __forceinline__ int vswz(int d) { return (d >> 1) & 7; }

// key of S-tile tau, tile row rho within a 64-key stage: the eight keys a lane group
// holds for one PV k-step are then consecutive.
__device__ __forceinline__ int stage_key(int tau, int rho) {
    return 32 * (tau >> 1) + 8 * (rho >> 2) + 4 * (tau & 1) + (rho & 3);
}

// 16 bytes per lane from global memory to LDS at byte `dst` + 16 * lane (dst uniform).  Inline assembly: the
// compiler waits for every such load before any later LDS read, which would take the stages one by one.
// It has no register result; stage_wait() and a barrier stand between it and the reads.
// ONCE: nobody reads the bytes again before they leave the caches, which the load passes by.
template <bool ONCE>
__device__ __forceinline__ void load_to_lds(const void* src, uint32_t dst) {
    if constexpr (ONCE)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(dst), "v"(src) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory", "m0");
}
// at most N vector memory operations of this wavefront still under way
template <int N>
__device__ __forceinline__ void stage_wait() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// max (or sum) over the lanes r, r+16, r+32, r+48, in every lane
__device__ __forceinline__ float rows_max(float v) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// committed length of sequence b as the attention reads it: clamped to [0, max_len]
__device__ __forceinline__ int attn_length(const AttnArgs& a, int b) {
    const int p = a.lengths[b];
    return p < 0 ? 0 : (p > a.max_len ? a.max_len : p);
}
// work items of one KV head of a sequence with committed length P (batches): its prefix splits, the last of
// which takes the block part along
__device__ __forceinline__ int attn_items(const AttnArgs& a, int P) { return max(1, (P + a.chunk - 1) / a.chunk); }

// Length-aware work item `item` -> (unit, split); false past the last item.  Wavefront 0 scans the
// sequences' item counts 64 at a time; the result goes to every thread through LDS.
__device__ bool attn_item(const AttnArgs& a, int item, int* unit, int* split) {
    __shared__ int su_s, ss_s;
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int base = 0, su = -1, ss = 0;
        for (int b0 = 0; b0 < a.n_seq && su < 0; b0 += 64) {
            const int b = b0 + lane;
            const int ni = b < a.n_seq ? attn_items(a, attn_length(a, b)) : 0;
            const int cnt = ni * a.n_kv_heads;
            int incl = cnt;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int t = __shfl_up(incl, off);
                if (lane >= off) incl += t;
            }
            const int excl = incl - cnt;
            const bool mine = cnt > 0 && item >= base + excl && item < base + incl;
            const unsigned long long who = __ballot(mine);
            if (who) {
                const int src = __ffsll((long long)who) - 1;
                const int r = __shfl(item - base - excl, src), nis = __shfl(ni, src);
                su = (b0 + src) * a.n_kv_heads + r / nis;
                ss = r % nis;
            }
            base += __shfl(incl, 63);
        }
        if (lane == 0) {
            su_s = su;
            ss_s = ss;
        }
    }
    __syncthreads();
    *unit = su_s;
    *split = ss_s;
    return su_s >= 0;
}

template <int D, int KH, int NS>
__global__ void __launch_bounds__(KH == 2 ? 512 : 768) __attribute__((amdgpu_waves_per_eu(KH == 2 && NS == 2 ? 4 : 1)))
attention_kernel(AttnArgs a) {
    typedef AttnCfg<D> C;
    constexpr int DC = D / 32;
    constexpr int DT = D / 16;
    constexpr int TPW = 4 / KH;                // S tiles (16 keys) per wavefront per stage
    // stage slots, each K tile (KCHUNKS) followed by the V tile (VCHUNKS)
    __shared__ uint4 lds[NS * C::CHUNKS];

    NLD_TS(TL_ATTENTION, 0);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const int r = lane & 15, g = lane >> 4;
    const int RZ = nw / KH;                    // row tiles per workgroup
    int split = blockIdx.x, unit = blockIdx.y;
    if (a.items) {
        if (!attn_item(a, blockIdx.x, &unit, &split)) return;   // the whole workgroup leaves
        unit = __builtin_amdgcn_readfirstlane(unit);
        split = __builtin_amdgcn_readfirstlane(split);
    }
    const int nkv = a.n_kv_heads, G = a.n_q_heads / nkv;
    const int b = unit / nkv;
    const int k = a.k_blk, R = G * k;
    const int kh = KH == 2 ? wave / RZ : 0;    // which half of each stage's keys
    const int rt = blockIdx.z * RZ + wave % RZ;
    const bool computes = rt < a.row_tiles;
    const int row = rt * 16 + r;
    const bool row_ok = computes && row < R;
    const int j = row_ok ? row % k : 0;

    const int P_raw = a.lengths[b];   // requested first; the loads below do not depend on it
    // Block columns this row sees: c <= lim and, in the quadratic layout, [lo_c, lo_c + n_c).  Verify: c <= j.
    // Draft: every column from row bidir_from on.  Quadratic layout (mode 2, chain length qk): chain row j sees
    // chain columns c <= j; a mask of group grp sees chain columns c <= grp and the columns of its own group.
    const int qk = a.quad_k;
    const bool qmask = a.mode == 2 && j >= qk;
    const int grp = qmask ? (j - qk) / qk : 0;
    const int lim = qmask ? grp : (a.mode == 1 && j >= a.bidir_from ? k : j);
    const int lo_c = qmask ? qk + grp * qk : 0, n_c = qmask ? qk : 0;

    const size_t head_off = (size_t)unit * a.max_len * D;
    const uint16_t* kbase = a.kc + head_off;
    const uint16_t* vbase = a.vc + head_off;
    const uint16_t* bkbase = a.blk_k + (size_t)unit * 2 * 64 * D;   // the block's keys and values: hi, then lo
    const uint16_t* bvbase = a.blk_v + (size_t)unit * 2 * 64 * D;

    // 64 keys from kp and vp into a slot: wavefront w takes 1 KiB blocks w, w + nw, ...  LDS position p of a
    // row holds chunk p ^ swizzle(row).
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
    // A batch's cache is read once per pass where one workgroup takes all rows (KH 2, NS 2: the batches' kernel
    // for up to 64 rows).  Non-temporal loads there: attention and merge 197 -> 183 us at batch 100, k = 1 (840 MB of
    // keys and values), 178 -> 160 us at batch 32, k = 16 (580 MB), 112 -> 104 us at batch 8 of 16000 keys.  With
    // five and more row tiles (KH 1) the matrix units are the bound, and one sequence's cache fits the caches:
    // neither gains.  (K and V rows requested half a stage apart, so that a stage and a half is always under
    // way: no gain over this, 241 instead of 210 us at KH 1.)
    constexpr bool ONCE = KH == 2 && NS == 2;
    auto dma = [&](const uint16_t* kp, const uint16_t* vp, int slot) __attribute__((always_inline)) {
        const uint32_t dst = lds0 + (uint32_t)slot * C::CHUNKS * 16;
#pragma unroll 1
        for (int i = wave; i < C::KCHUNKS / 64; i += nw) {
            const int q = i * 64 + lane, kr = q / C::KCH, c = (q % C::KCH) ^ kswz<D>(kr);
            load_to_lds<ONCE>(kp + (kr * C::KCH + c) * 8, __builtin_amdgcn_readfirstlane(dst + i * 1024));
        }
#pragma unroll 1
        for (int i = wave; i < C::VCHUNKS / 64; i += nw) {
            const int q = i * 64 + lane, d = q >> 3, c = (q & 7) ^ vswz(d);
            load_to_lds<ONCE>(vp + (d * 8 + c) * 8, __builtin_amdgcn_readfirstlane(dst + C::KCHUNKS * 16 + i * 1024));
        }
    };
    auto dma_keys = [&](int kb, int slot) __attribute__((always_inline)) {
        dma(kbase + (size_t)kb * D, vbase + (size_t)kb * D, slot);   // kb is a multiple of 64: a V tile's start
    };
    constexpr int PB = C::BLOCKS / 8;   // a wavefront's loads per stage (NS > 2 runs with 8 wavefronts)

    // Operand positions in LDS: K chunk c of S tile tau at kidx[c] + tau's rows, V rows of 16 dims apart.
    // (The swizzles only see row bits that tau and the dim tile leave alone.)
    int kidx[DC], vidx[TPW / 2];
    {
        const int kr = stage_key(TPW * kh, r);
#pragma unroll
        for (int c = 0; c < DC; ++c) kidx[c] = kr * C::KCH + ((4 * c + g) ^ kswz<D>(kr));
#pragma unroll
        for (int kk = 0; kk < TPW / 2; ++kk) vidx[kk] = C::KCHUNKS + r * 8 + ((4 * ((TPW / 2) * kh + kk) + g) ^ vswz(r));
    }

    // The first stage is requested before the committed length is known: a prefix split's first 64 keys
    // (always inside the cache; masked below if they are not committed), or the block part's hi halves.
    const bool blockonly = !a.items && split == a.n_splits;
    int split_beg = split * a.chunk;   // prefix splits: first key of the split (< max_len)
    if (blockonly) dma(bkbase, bvbase, 0);
    else dma_keys(split_beg, 0);

    const uint4 zero4 = {0u, 0u, 0u, 0u};
    uint4 qb[DC], ql[DC];   // split queries: hi and lo operands
    {
        const uint16_t* qp = a.q + ((size_t)((unit * a.row_tiles + rt) * DC * 2) * 64 + lane) * 8;
#pragma unroll
        for (int c = 0; c < DC; ++c) {
            qb[c] = row_ok ? *(const uint4*)(qp + (size_t)c * 1024) : zero4;
            ql[c] = row_ok ? *(const uint4*)(qp + (size_t)c * 1024 + SPLIT_LO) : zero4;
        }
    }

    const int P = P_raw < 0 ? 0 : (P_raw > a.max_len ? a.max_len : P_raw);
    // One sequence: the n_splits prefix splits are cut from the committed length, chunk = ceil(P / n_splits)
    // rounded up to whole stages (at most the plan's chunk, which was cut from max_len), so that a cache much
    // longer than its prefix still spreads the prefix over every split.  The first stage went out at the
    // plan's split start; it is requested again where the two differ.
    int chunk = a.chunk;
    if (!a.items && !blockonly) {
        chunk = max(64, ((P + a.n_splits - 1) / a.n_splits + 63) / 64 * 64);
        const int beg = split * chunk;
        if (beg != split_beg) {
            split_beg = beg;
            if (beg < P) {   // beg < P <= max_len, a multiple of 64: inside the cache
                stage_wait<0>();   // the two requests write the same slot
                dma_keys(beg, 0);
            }
        }
    }
    // committed keys [split_beg, kend) of [0, P), then (the unit's last item, or the block's own workgroup)
    // the block's keys [P, P + k)
    const int kend = min(split_beg + chunk, P);
    const int nst = blockonly ? 0 : (kend > split_beg ? (kend - split_beg + 63) / 64 : 0);
    const bool blockpart = blockonly || (a.items && split == attn_items(a, P) - 1);
    NLD_TS(TL_ATTENTION, 1);   // committed length known

    f32x4_t acc[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    // p = exp2(s - m_ref), m_ref the largest score so far, so that the largest p is 1 and loses nothing in its
    // split, however long the item; the denominator sums the split p (ones against P^T on MFMA), so that what the
    // others lose cancels in a peaked row.  A reference that lags the maximum by up to 2^8 rescales less often, but
    // costs precision where items are long: error of the logits behind one layer 8.75e-6 against 8.35e-6 for 8
    // sequences of 16 rows, 11.1e-6 against 10.5e-6 for 4 of 32 rows of the 14B shapes.  Passes of 56 to 512 rows
    // take the same time either way within 0.5%.
    float m_ref = -INFINITY;
    // In a batch the reference also goes down to a stage's own maximum, by up to 2^8 a stage while the row's sum is
    // below 2^12 (so weights stay below 2^20): the largest weight of every stage is then exact, as if each stage were an
    // item.  Errors of the logits behind one layer with items of 64 keys / of 384 without it / with it: 7.85, 7.95 and
    // 7.83e-6 (8 sequences of 2 rows), 8.29, 8.38 and 8.28e-6 (8 of 16 rows).  Passes take 0 to 0.3% longer.  With
    // five and more row tiles it stays out of items of 1024 keys, which come in at the old error without it (9.7 against
    // 9.9e-6, 10 sequences of 26 rows, 14B shapes) and would take 1.2% longer (a pass of 8 sequences of 32 rows and 16384
    // keys 2702 against 2669 us).
    const float drop = NS == 2 && (KH == 2 || (a.items && a.chunk < 1024)) ? 8.f : 0.f;
    f32x4_t l4 = {0.f, 0.f, 0.f, 0.f};   // the row's sum, four times

    // One stage of keys kb .. kb+63 from slot hi; own: the block part, its keys' and values' lo halves in slot
    // lo; edge: the stage holds keys at or past `end` (or the block's), which are masked.
    auto stage = [&](int kb, int end, int hi, int lo, auto own, auto edge) __attribute__((always_inline)) {
        const uint4* kv = lds + hi * C::CHUNKS;
        const uint4* kvl = lds + lo * C::CHUNKS;
        f32x4_t s[TPW];
#pragma unroll
        for (int tt = 0; tt < TPW; ++tt) s[tt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        // A tile's products with the lo halves (2^-8 of the score) come first, so that only the hi products round
        // at the score's size, as with two accumulators and without the second one's registers.
        // The scheduling barriers keep the compiler from reading a whole stage's operands ahead, which takes
        // more registers than a wavefront has here.
#pragma unroll
        for (int tt = 0; tt < TPW; ++tt) {
            const int row = (32 * (tt >> 1) + 4 * (tt & 1)) * C::KCH;
            uint4 kop[DC];
#pragma unroll
            for (int c = 0; c < DC; ++c) kop[c] = kv[kidx[c] + row];
#pragma unroll
            for (int c = 0; c < DC; ++c) {
                s[tt] = mfma_16x16x32(kop[c], ql[c], s[tt]);
                if constexpr (own) s[tt] = mfma_16x16x32(kvl[kidx[c] + row], qb[c], s[tt]);
            }
#pragma unroll
            for (int c = 0; c < DC; ++c) s[tt] = mfma_16x16x32(kop[c], qb[c], s[tt]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (edge) {
#pragma unroll
            for (int tt = 0; tt < TPW; ++tt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int key = kb + stage_key(TPW * kh + tt, 4 * g + i);
                    const int c = key - P;   // block column (negative: the prefix)
                    const bool vis = (key < end) & ((c <= lim) | ((unsigned)(c - lo_c) < (unsigned)n_c));
                    s[tt][i] = vis ? s[tt][i] : -INFINITY;
                }
        }
        __builtin_amdgcn_sched_barrier(0);
        float mloc = s[0][0];
#pragma unroll
        for (int tt = 0; tt < TPW; ++tt)
#pragma unroll
            for (int i = 0; i < 4; ++i) mloc = fmaxf(mloc, s[tt][i]);
        mloc = rows_max(mloc) * a.scale_log2;      // scale_log2 > 0
        const float m_new = fmaxf(mloc, l4[0] < 4096.f ? m_ref - drop : m_ref);
        if (m_new != m_ref) {                      // new reference: rescale what has accumulated
            const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);   // 0 when m_ref = -inf
            l4 *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) acc[dt] *= alpha;
            m_ref = m_new;
        }
        const float m_use = m_ref == -INFINITY ? 0.f : m_ref;   // no key visible yet: every p is exp2(-inf) = 0
        float p[4 * TPW];
#pragma unroll
        for (int e = 0; e < 4 * TPW; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(s[e >> 2][e & 3], a.scale_log2, -m_use));
#pragma unroll
        for (int kk = 0; kk < TPW / 2; ++kk) {
            // slot jj of lane group g <-> key kb + 32ks + 8g + jj
            uint4 pop, pol;                               // P^T as split operands
            split8(p + 8 * kk, pop, pol, a.plain & SITE_P);
            const uint4 ones = {0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
            l4 = mfma_16x16x32(ones, pol, l4);
            l4 = mfma_16x16x32(ones, pop, l4);
            const int key0 = kb + 32 * ((TPW / 2) * kh + kk) + 8 * g;
            uint32_t vm[4];                               // V rows past the valid keys may hold anything
#pragma unroll
            for (int e = 0; e < 4; ++e)
                vm[e] = (key0 + 2 * e < end ? 0xFFFFu : 0u) | (key0 + 2 * e + 1 < end ? 0xFFFF0000u : 0u);
            auto masked = [&](uint4 v) __attribute__((always_inline)) {
                return edge ? uint4{v.x & vm[0], v.y & vm[1], v.z & vm[2], v.w & vm[3]} : v;
            };
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const int at = vidx[kk] + dt * 128;
                const uint4 vop = masked(kv[at]);
                acc[dt] = mfma_16x16x32(vop, pop, acc[dt]);
                acc[dt] = mfma_16x16x32(vop, pol, acc[dt]);
                if constexpr (own) acc[dt] = mfma_16x16x32(masked(kvl[at]), pop, acc[dt]);
                if ((dt & 3) == 3 || own) __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    struct Yes { constexpr operator bool() const { return true; } };
    struct No { constexpr operator bool() const { return false; } };
    const int nfull = kend > split_beg ? (kend - split_beg) / 64 : 0;   // whole stages; the rest masks keys

    // Stage st is multiplied from slot st % NS.  NS = 2: the next one (then the block's hi halves) is under way
    // meanwhile.  NS = 4 (one sequence): stages 1 .. 3 are requested once the first is in LDS, since
    // requested with it they arrive interleaved and the first comes late, and three stay under way.
    // The queries are named here so that the compiler's own wait for their loads stands here too: it does not
    // know of the wait before, and in the loop that wait would also be one for every stage under way.
    stage_wait<0>();
#pragma unroll
    for (int c = 0; c < DC; ++c) {
        asm volatile("" : "+v"(qb[c].x), "+v"(qb[c].y), "+v"(qb[c].z), "+v"(qb[c].w));
        asm volatile("" : "+v"(ql[c].x), "+v"(ql[c].y), "+v"(ql[c].z), "+v"(ql[c].w));
    }
    __syncthreads();
    NLD_TS(TL_ATTENTION, 2);   // first stage in LDS
    if constexpr (NS == 4) {
#pragma unroll
        for (int i = 1; i < 4; ++i)
            if (i < nst) dma_keys(split_beg + 64 * i, i);
        auto next = [&](int st) __attribute__((always_inline)) {   // stage st done: st + 1 has to be in LDS
            const int ahead = min(nst - 1 - st, 3) - 1;   // stages under way after it
            if (ahead >= 2) stage_wait<2 * PB>();
            else if (ahead == 1) stage_wait<PB>();
            else stage_wait<0>();
            __syncthreads();
            if (st + 4 < nst) dma_keys(split_beg + 64 * (st + 4), st % 4);
        };
        for (int st = 0; st < nfull; ++st) {
            if (computes) stage(split_beg + 64 * st, kend, st % 4, 0, No{}, No{});
            next(st);
        }
        if (nst > nfull) {
            if (computes) stage(split_beg + 64 * nfull, kend, nfull % 4, 0, No{}, Yes{});
            next(nfull);
        }
    } else {
        auto ahead = [&](int st) __attribute__((always_inline)) {   // what follows stage st, into the other slot
            if (st + 1 < nst) dma_keys(split_beg + 64 * (st + 1), (st + 1) & 1);
            else if (blockpart) dma(bkbase, bvbase, (st + 1) & 1);
        };
        for (int st = 0; st < nfull; ++st) {
            ahead(st);
            if (computes) stage(split_beg + 64 * st, kend, st & 1, 0, No{}, No{});
            stage_wait<0>();
            __syncthreads();
        }
        if (nst > nfull) {
            ahead(nfull);
            if (computes) stage(split_beg + 64 * nfull, kend, nfull & 1, 0, No{}, Yes{});
            stage_wait<0>();
            __syncthreads();
        }
    }
    if (blockpart) {
        const int hi = nst % NS;   // NS = 4: the block's own workgroup, nst = 0
        if (!blockonly && nst == 0) dma(bkbase, bvbase, hi);   // no prefix: slot 0 holds uncommitted keys
        dma(bkbase + 64 * D, bvbase + 64 * D, hi ^ 1);
        stage_wait<0>();
        __syncthreads();
        if (computes) stage(P, P + k, hi, hi ^ 1, Yes{}, Yes{});
        __syncthreads();
    }

    NLD_TS(TL_ATTENTION, 3);   // stages done
    float l_tot = l4[0];
    if constexpr (KH == 2) {
        // merge the two key halves of each row tile through LDS (the stage buffers are free now)
        float* mrg = (float*)lds;                    // [RZ][16 rows][D + 2] floats, within the stage slots
        float* slot = mrg + ((size_t)(wave % RZ) * 16 + r) * (D + 2);
        if (kh == 1 && computes) {
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int i = 0; i < 4; ++i) slot[16 * dt + 4 * g + i] = acc[dt][i];
            if (g == 0) {
                slot[D] = m_ref;
                slot[D + 1] = l_tot;
            }
        }
        __syncthreads();
        if (kh == 1 || !computes) return;
        const float m2 = slot[D], l2 = slot[D + 1];
        const float mm = fmaxf(m_ref, m2);
        const float w1 = (m_ref == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m_ref - mm);
        const float w2 = (m2 == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m2 - mm);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[dt][i] = acc[dt][i] * w1 + slot[16 * dt + 4 * g + i] * w2;
        l_tot = l_tot * w1 + l2 * w2;
        m_ref = mm;
    }
    if (!computes) return;
    const size_t pbase = ((size_t)unit * a.n_parts + split) * a.rows_pad + row;
    float* po = a.part_o + pbase * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) *(float4*)(po + 16 * dt + 4 * g) = float4{acc[dt][0], acc[dt][1], acc[dt][2], acc[dt][3]};
    if (g == 0) *(float2*)(a.part_ml + pbase * 2) = float2{m_ref, l_tot};
#ifdef NLD_TIMELINE
    __syncthreads();
#endif
    NLD_TS(TL_ATTENTION, 4);
}

// Merge of the partials (prefix splits + block part): one workgroup per (unit, query
// row), one thread per head dim; writes the split attention output.
template <int D>
__global__ void __launch_bounds__(D) attention_combine_kernel(AttnArgs a) {
    __shared__ float wsh[256];
    __shared__ float inv_den;
    NLD_TS(TL_COMBINE, 0);
    const int unit = blockIdx.x, rw = blockIdx.y, d = threadIdx.x;
    const int nkv = a.n_kv_heads, G = a.n_q_heads / nkv;
    const int b = unit / nkv, kvh = unit % nkv, k = a.k_blk;
    // parts: a batch's work items, or one sequence's prefix splits and the block part
    const int ns = a.items ? attn_items(a, attn_length(a, b)) : a.n_splits + 1;
    const size_t ubase = (size_t)unit * a.n_parts * a.rows_pad + rw;
    // With at most FAST parts every load of the workgroup is issued at once: thread d's part
    // statistics and its column of every part's output.  More parts take the looped path.
    constexpr int FAST = 32;
    const bool fast = ns <= FAST;
    float2 ml0 = float2{-INFINITY, 0.f};
    float os[FAST];
    if (fast) {
        if (d < ns) ml0 = *(const float2*)(a.part_ml + (ubase + (size_t)d * a.rows_pad) * 2);
#pragma unroll
        for (int e = 0; e < FAST; ++e)
            os[e] = e < ns ? a.part_o[(ubase + (size_t)e * a.rows_pad) * D + d] : 0.f;
    }
    // split statistics -> weights exp2(m_s - max) in LDS (ns <= 256)
    float ms = -INFINITY, ls = 0.f;
    if (fast) {
        if (d < ns) wsh[d] = ml0.x;
        ms = ml0.x;
    } else {
        for (int sp = d; sp < ns; sp += D) {
            const float2 ml = *(const float2*)(a.part_ml + (ubase + (size_t)sp * a.rows_pad) * 2);
            wsh[sp] = ml.x;
            ms = fmaxf(ms, ml.x);
        }
    }
    // block max over D threads (D <= 128: two wavefronts at most)
    ms = fmaxf(ms, __shfl_xor(ms, 32));
    ms = fmaxf(ms, __shfl_xor(ms, 16));
    ms = fmaxf(ms, __shfl_xor(ms, 8));
    ms = fmaxf(ms, __shfl_xor(ms, 4));
    ms = fmaxf(ms, __shfl_xor(ms, 2));
    ms = fmaxf(ms, __shfl_xor(ms, 1));
    __shared__ float wmax[2];
    if ((d & 63) == 0) wmax[d >> 6] = ms;
    __syncthreads();
    const float mx = (D > 64) ? fmaxf(wmax[0], wmax[1]) : wmax[0];
    if (fast) {
        if (d < ns) {
            const float w = (ml0.x == -INFINITY) ? 0.f : exp2f(ml0.x - mx);
            ls = w * ml0.y;
            wsh[d] = w;
        }
    } else {
        for (int sp = d; sp < ns; sp += D) {
            const float msp = wsh[sp];
            const float w = (msp == -INFINITY) ? 0.f : exp2f(msp - mx);
            ls += w * a.part_ml[(ubase + (size_t)sp * a.rows_pad) * 2 + 1];
            wsh[sp] = w;
        }
    }
    ls += __shfl_xor(ls, 32);
    ls += __shfl_xor(ls, 16);
    ls += __shfl_xor(ls, 8);
    ls += __shfl_xor(ls, 4);
    ls += __shfl_xor(ls, 2);
    ls += __shfl_xor(ls, 1);
    __shared__ float wden[2];
    if ((d & 63) == 0) wden[d >> 6] = ls;
    __syncthreads();
    if (d == 0) inv_den = 1.0f / ((D > 64) ? (wden[0] + wden[1]) : wden[0]);
    __syncthreads();
    // the parts in order, one product-sum each (the same order on both paths)
    float num = 0.f;
    if (fast) {
#pragma unroll
        for (int e = 0; e < FAST; ++e)
            if (e < ns) num += wsh[e] * os[e];
    } else {
        int sp = 0;
        for (; sp + 8 <= ns; sp += 8) {
            float o8[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) o8[e] = a.part_o[(ubase + (size_t)(sp + e) * a.rows_pad) * D + d];
#pragma unroll
            for (int e = 0; e < 8; ++e) num += wsh[sp + e] * o8[e];
        }
        for (; sp < ns; ++sp) num += wsh[sp] * a.part_o[(ubase + (size_t)sp * a.rows_pad) * D + d];
    }
    const int hl = rw / k, j = rw % k;
    store_split(a.o, split_index(b * k + j, (kvh * G + hl) * D + d, a.n_q_heads * D / 32), num * inv_den,
                a.plain & SITE_O);
    NLD_TS(TL_COMBINE, 1);
}

// The same merge where there are rows for at least 512 workgroups of 256 threads: D / 8 lanes take a row, 8 dims
// each, so that partials come and the split output goes in 16-byte pieces, four parts at a time under a running
// maximum, without LDS.  Bound by the partials' reads: 17.9 -> 9.7 us at 16384 rows (256 units of 64), 14.6 ->
// 14.1 us at 10240 rows of 17 parts (89 MB).  Below that the kernel above has more loads under way: 5.9 against
// 8.7 us at 3840 rows, 4.7 against 4.8 us at 512 rows of one sequence (with the parts shared by eight groups).
template <int D>
__global__ void __launch_bounds__(256) attention_combine_rows_kernel(AttnArgs a, int rows) {
    constexpr int LP = D / 8, RW = 256 / LP;   // lanes per row, rows per workgroup
    constexpr int U = 4;                        // parts under way
    NLD_TS(TL_COMBINE, 0);
    const int c = threadIdx.x % LP;
    const int unit = blockIdx.x, rw = blockIdx.y * RW + threadIdx.x / LP;
    if (rw >= rows) return;
    const int nkv = a.n_kv_heads, G = a.n_q_heads / nkv;
    const int b = unit / nkv, kvh = unit % nkv, k = a.k_blk;
    const int ns = a.items ? attn_items(a, attn_length(a, b)) : a.n_splits + 1;
    const size_t base = (size_t)unit * a.n_parts * a.rows_pad + rw;

    float m = -INFINITY, l = 0.f, o[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = 0.f;
    for (int e0 = 0; e0 < ns; e0 += U) {
        float2 ml[U];
        float4 v[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ml[u] = float2{-INFINITY, 0.f};
            v[u][0] = v[u][1] = float4{0.f, 0.f, 0.f, 0.f};
            if (e0 + u < ns) {
                const size_t at = base + (size_t)(e0 + u) * a.rows_pad;
                ml[u] = *(const float2*)(a.part_ml + at * 2);
                v[u][0] = *(const float4*)(a.part_o + at * D + 8 * c);
                v[u][1] = *(const float4*)(a.part_o + at * D + 8 * c + 4);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float mm = fmaxf(m, ml[u].x);
            const float w0 = m == -INFINITY ? 0.f : exp2f(m - mm), w1 = ml[u].x == -INFINITY ? 0.f : exp2f(ml[u].x - mm);
            const float op[8] = {v[u][0].x, v[u][0].y, v[u][0].z, v[u][0].w, v[u][1].x, v[u][1].y, v[u][1].z, v[u][1].w};
            l = l * w0 + ml[u].y * w1;
#pragma unroll
            for (int i = 0; i < 8; ++i) o[i] = o[i] * w0 + op[i] * w1;
            m = mm;
        }
    }
    const float inv = 1.0f / l;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] *= inv;
    uint4 hi, lo;
    split8(o, hi, lo, a.plain & SITE_O);
    uint16_t* out = a.o + split_index(b * k + rw % k, (kvh * G + rw / k) * D + 8 * c, a.n_q_heads * D / 32);
    *(uint4*)out = hi;
    *(uint4*)(out + SPLIT_LO) = lo;
    NLD_TS(TL_COMBINE, 1);
}

template <int D>
static hipError_t launch_attention_d(int kh, int waves, dim3 grid, const AttnArgs& a, hipStream_t s) {
    const dim3 blk(64 * waves);
    if (kh == 2 && !a.items) launch(attention_kernel<D, 2, 4>, grid, blk, s, a);
    else if (kh == 2) launch(attention_kernel<D, 2, 2>, grid, blk, s, a);
    else launch(attention_kernel<D, 1, 2>, grid, blk, s, a);
    return hipGetLastError();
}

hipError_t launch_attention(int head_dim, int kh, int waves, int zslices, int units, const AttnArgs& a, hipStream_t s) {
    // four stage slots count on 8 wavefronts' loads
    if (waves < kh || waves % kh || waves > (kh == 2 ? 8 : 12) || (kh == 2 && !a.items && waves != 8)) return hipErrorInvalidValue;
    // prefix splits + the block part per unit; length-aware items: all of them on x
    const dim3 grid = a.items ? dim3(a.n_splits * units, 1, zslices) : dim3(a.n_splits + 1, units, zslices);
    return head_dim == 128 ? launch_attention_d<128>(kh, waves, grid, a, s) : launch_attention_d<64>(kh, waves, grid, a, s);
}

template <int D>
static hipError_t launch_combine_d(int units, int rows, const AttnArgs& a, hipStream_t s) {
    const dim3 wide(units, (rows + 2048 / D - 1) / (2048 / D));   // 2048 / D rows per workgroup
    if ((size_t)wide.x * wide.y >= 512) launch(attention_combine_rows_kernel<D>, wide, dim3(256), s, a, rows);
    else launch(attention_combine_kernel<D>, dim3(units, rows), dim3(D), s, a);
    return hipGetLastError();
}

hipError_t launch_attention_combine(int head_dim, int units, int rows, const AttnArgs& a, hipStream_t s) {
    return head_dim == 128 ? launch_combine_d<128>(units, rows, a, s) : launch_combine_d<64>(units, rows, a, s);
}

// =====================================================================================
// Embedding gather of the block (block assembly per call kind) into the fp32 residual.
// =====================================================================================
__global__ void __launch_bounds__(256) embed_kernel(EmbedArgs a) {
    const int m = blockIdx.x;
    const int b = m / a.k_blk, j = m % a.k_blk;
    if (m == 0)
        for (int i = threadIdx.x; i < a.n_tile_ctr; i += blockDim.x) a.tile_ctr[i] = 0u;
    if (a.keys)
        for (int i = threadIdx.x; i < KEY_SLOTS; i += blockDim.x) a.keys[(size_t)m * KEY_SLOTS + i] = 0ull;
    // RoPE table of this row (used by every layer's QKV epilogue): angle pos * theta_i
    // reduced to [-pi, pi] and evaluated in fp64, stored as fp32 (cos, sin).
    if ((int)threadIdx.x < a.head_dim / 2) {
        const int fi = threadIdx.x;
        // quadratic layout: mask r of group c (row qk + c*qk + r - 1) sits at P + c + r
        const int qk = a.quad_k;
        const int off = (qk > 0 && j >= qk) ? (j - qk) / qk + (j - qk) % qk + 1 : j;
        const int pos = committed_length(a.lengths, b, a.max_len, a.status) + off;
        const double two_pi = 6.283185307179586476925286766559;
        double ang = (double)pos * a.inv_freq[fi];
        ang -= two_pi * rint(ang * (1.0 / two_pi));
        a.rope[(size_t)m * (a.head_dim / 2) + fi] = float2{(float)cos(ang), (float)sin(ang)};
    }
    int tok;
    if (a.source == 0) tok = a.tokens[m];
    else if (j == 0) tok = a.anchor[b];
    else if (a.source == 1) tok = a.mask_id;
    else if (a.source == 3) tok = j < a.quad_k ? a.draft[b * (a.quad_k - 1) + j - 1] : a.mask_id;
    else tok = a.draft[b * (a.k_blk - 1) + j - 1];
    if (tok < 0 || tok >= a.vocab) {
        if (threadIdx.x == 0) atomicOr(a.status, DEV_BAD_TOKEN);
        tok = 0;
    }
    const uint16_t* e = a.embed + (size_t)tok * a.hidden;
    const size_t row = (size_t)m * a.hidden;
    const int chunks = a.hidden / 16;
    float row_ss = 0.f;
    for (int c = threadIdx.x; c < chunks; c += blockDim.x) {   // 16 columns per thread
        float ss = 0.f;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int col = 16 * c + 8 * h;
            const uint4 w = *(const uint4*)(e + col);
            const uint4 gg = *(const uint4*)(a.gain + col);
            const uint32_t ew[4] = {w.x, w.y, w.z, w.w}, gw[4] = {gg.x, gg.y, gg.z, gg.w};
            float xv[8], xgv[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                xv[2 * q] = bf16_to_f32(ew[q] & 0xFFFFu);
                xv[2 * q + 1] = bf16_to_f32(ew[q] >> 16);
                xgv[2 * q] = xv[2 * q] * bf16_to_f32(gw[q] & 0xFFFFu);
                xgv[2 * q + 1] = xv[2 * q + 1] * bf16_to_f32(gw[q] >> 16);
            }
#pragma unroll
            for (int q = 0; q < 8; ++q) ss += xv[q] * xv[q];
            *(float4*)(a.x + row + col) = float4{xv[0], xv[1], xv[2], xv[3]};
            *(float4*)(a.x + row + col + 4) = float4{xv[4], xv[5], xv[6], xv[7]};
            uint4 hi, lo;
            split8(xgv, hi, lo, a.plain & SITE_NORM);
            const size_t xi = split_index(m, col, a.hidden / 32);
            *(uint4*)(a.xg + xi) = hi;
            *(uint4*)(a.xg + xi + SPLIT_LO) = lo;
        }
        row_ss += ss;
    }
    row_ss = wave_sum(row_ss);
    const int sums = embed_sums(a.hidden), wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0 && wave < sums) a.part_ss[(size_t)m * sums + wave] = row_ss;
}

hipError_t launch_embed(const EmbedArgs& a, hipStream_t s) {
    launch(embed_kernel, dim3(a.M), dim3(64 * EMBED_WAVES), s, a);
    return hipGetLastError();
}

// =====================================================================================
// Per-sequence finish: argmax of each block row (from the LM head's per-workgroup
// keys, or from given logits; lowest index among equal maxima), then draft
// extraction (d_j = argmax of draft row j), longest-prefix acceptance with the
// bonus token and the commit of L+1 rows, or a denoising step's commit: masked
// rows whose top-1 softmax probability exceeds the threshold take their argmax,
// else the most confident masked row does.  A refresh only commits k-1 rows.
// One workgroup per sequence, one wavefront per row.
// =====================================================================================
// the float value an argmax key was made from
__device__ __forceinline__ float argmax_key_value(unsigned long long key) {
    const uint32_t ord = (uint32_t)(key >> 32);
    return __uint_as_float((ord & 0x80000000u) ? (ord ^ 0x80000000u) : ~ord);
}

// max over the wavefront, in every lane: register moves within the rows of 16 lanes, then across them
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = max(v, row_ror<8>(v));
    v = max(v, row_ror<4>(v));
    v = max(v, row_ror<2>(v));
    v = max(v, row_ror<1>(v));
    const auto a = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    v = max((uint32_t)a[0], (uint32_t)a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return max((uint32_t)b[0], (uint32_t)b[1]);
}
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, row_ror<8>(v));
    v = fmaxf(v, row_ror<4>(v));
    v = fmaxf(v, row_ror<2>(v));
    return rows_max(fmaxf(v, row_ror<1>(v)));
}
__device__ __forceinline__ unsigned long long wave_max_key(unsigned long long key) {
    const uint32_t ord = (uint32_t)(key >> 32), top = wave_max_u32(ord);
    return ((unsigned long long)top << 32) | wave_max_u32(ord == top ? (uint32_t)key : 0u);
}

// A row's LM-head partials, a lane taking every 64th.  The panel GEMM leaves one per column group, 792 for the 8B
// vocabulary, where the normed GEMM leaves one per CU.  Eight loads a row are under way per lane, through a buffer
// descriptor that ends with the row (past it: zeros, the empty key and an empty sum, without a branch or an address per
// load), and the softmax sums take the maximum of a round first.  A finish runs once a pass, from a cold instruction
// cache, so short code counts as much: sixteen loads ahead took 8.2 us at 32 rows.  One load and one merge after the
// other the quadratic finish took 7.8 us and the ensemble 12.0 (8B vocabulary, chain length 7), now 4.9 and 8.1; the
// finish of 32 rows took 6.6 us and now 6.1, of a denoising step 27.1 and now 14.6.
constexpr int PARTS_AHEAD = 8;
struct PartRow {
    __amdgpu_buffer_rsrc_t rs;
    // base uniform; on = false: an empty row
    __device__ __forceinline__ PartRow(const void* base, int n, bool on) {
        rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, on ? 8 * n : 0, 0x00027000);
    }
    __device__ __forceinline__ uint2 load(int p) const {
        typedef uint32_t u32x2_b __attribute__((ext_vector_type(2)));
        const u32x2_b v = __builtin_bit_cast(u32x2_b, __builtin_amdgcn_raw_buffer_load_b64(rs, 8 * p, 0, 0));
        return uint2{v[0], v[1]};
    }
};

// the argmax keys of rows m and m2 (m2 < 0: none, the empty key), in every lane of the wavefront
__device__ __forceinline__ void row_keys(const FinishArgs& a, int m, int m2, int lane, unsigned long long (&best)[2]) {
    const PartRow row[2] = {PartRow(a.part_keys + (size_t)m * a.n_keys, a.n_keys, true),
                            PartRow(a.part_keys + (size_t)max(m2, 0) * a.n_keys, a.n_keys, m2 >= 0)};
    best[0] = best[1] = 0ull;
    for (int p0 = lane; p0 - lane < a.n_keys; p0 += 64 * PARTS_AHEAD) {
        uint2 v[2][PARTS_AHEAD];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int u = 0; u < PARTS_AHEAD; ++u) v[q][u] = row[q].load(p0 + 64 * u);
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int u = 0; u < PARTS_AHEAD; ++u)
                best[q] = umax64(best[q], ((unsigned long long)v[q][u].y << 32) | v[q][u].x);
    }
    best[0] = wave_max_key(best[0]);
    best[1] = wave_max_key(best[1]);
}

// the softmax statistics (max, sum of exp(z - max)) of row m, in every lane of the wavefront; empty partials (a maximum
// of -inf, or past the row's end a sum of 0) take no part, as in lse_merge
__device__ __forceinline__ float2 row_lse(const FinishArgs& a, int m, int lane) {
    const PartRow row(a.part_lse + (size_t)m * a.n_parts, a.n_parts, true);
    float2 st = float2{-INFINITY, 0.f};
    for (int p0 = lane; p0 - lane < a.n_parts; p0 += 64 * PARTS_AHEAD) {
        float2 v[PARTS_AHEAD];
        float mx = -INFINITY, sum = 0.f;
#pragma unroll
        for (int u = 0; u < PARTS_AHEAD; ++u) {
            const uint2 w = row.load(p0 + 64 * u);
            v[u] = float2{__uint_as_float(w.x), __uint_as_float(w.y)};
        }
#pragma unroll
        for (int u = 0; u < PARTS_AHEAD; ++u) {
            if (v[u].y == 0.f) v[u].x = -INFINITY;
            mx = fmaxf(mx, v[u].x);
        }
        mx = wave_max(mx);
#pragma unroll
        for (int u = 0; u < PARTS_AHEAD; ++u) sum += v[u].x != -INFINITY ? v[u].y * expf(v[u].x - mx) : 0.f;
        st = lse_merge(st, float2{mx, wave_sum(sum)});
    }
    return st;
}

// Commit n more rows of sequence b.  Rows at or past max_len were never written (the QKV epilogue
// skipped them and set DEV_CAPACITY), so the length stops at max_len: every row below it is valid.
__device__ __forceinline__ void advance_length(const FinishArgs& a, int b, int n) {
    const int p = a.lengths[b] + n;
    if (p > a.max_len) {
        atomicOr(a.status, DEV_CAPACITY);
        a.lengths[b] = a.max_len;
    } else {
        a.lengths[b] = p;
    }
}

__global__ void __launch_bounds__(1024) finish_kernel(FinishArgs a) {
    __shared__ int32_t am[64], in_s[64];
    __shared__ float cf[64];
    const int b = blockIdx.x, k = a.k_blk;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    const bool denoise = a.finish == FINISH_DENOISE;
    if (a.finish == FINISH_REFRESH) {
        if (threadIdx.x != 0) return;
        const int32_t* blk = a.block + (size_t)b * k;
        for (int j = 1; j < k; ++j)
            if (blk[j] == a.mask_id) atomicOr(a.status, DEV_MASK_LEFT);
        a.next_anchor[b] = blk[k - 1];
        advance_length(a, b, k - 1);
        return;
    }
    // the block (denoising) or the drafts to accept, read beside the partials: one thread reading them one by one at the
    // end took longer than all the rest of a denoising finish
    const int32_t* in = denoise ? a.block + (size_t)b * k : a.draft_in + (size_t)b * (k - 1);
    if ((denoise || a.finish == FINISH_ACCEPT) && (int)threadIdx.x < (denoise ? k : k - 1)) in_s[threadIdx.x] = in[threadIdx.x];
    auto row_done = [&](int jr, unsigned long long best, float2 st) __attribute__((always_inline)) {
        if (lane != 0) return;
        const int m = b * k + jr, idx = argmax_key_index(best);
        am[jr] = idx;
        if (a.argmax_out) a.argmax_out[m] = idx;
        if (denoise) {
            // probability of the argmax token: exp(z_best - max) / sum (the max is z_best)
            const float c = expf(argmax_key_value(best) - st.x) / st.y;
            cf[jr] = c;
            if (a.conf_out) a.conf_out[m] = c;
        }
    };
    if (a.part_keys) {
        for (int jr = wave; jr < k; jr += 2 * nw) {   // two rows of a wavefront at a time
            const int m = b * k + jr, m2 = jr + nw < k ? m + nw : -1;
            unsigned long long best[2];
            row_keys(a, m, m2, lane, best);
#pragma unroll 1
            for (int q = 0; q < (m2 >= 0 ? 2 : 1); ++q) {
                float2 st = float2{-INFINITY, 0.f};
                if (denoise) st = row_lse(a, q ? m2 : m, lane);
                row_done(q ? jr + nw : jr, q ? best[1] : best[0], st);
            }
        }
    } else {   // from given logits
        const int excl = denoise ? a.mask_id : -1;
        for (int jr = wave; jr < k; jr += nw) {
            const float* lg = a.logits + (size_t)(b * k + jr) * a.vocab;
            unsigned long long best = 0ull;
            float2 st = float2{-INFINITY, 0.f};   // softmax statistics (denoising only)
            for (int n = lane; n < a.vocab; n += 64) {
                if (n == excl) continue;
                const float v = lg[n];
                best = umax64(best, argmax_key(v, (uint32_t)n));
                if (denoise) st = lse_merge(st, float2{v, 1.f});
            }
            best = wave_max_key(best);
            if (denoise) {
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) st = lse_merge(st, float2{__shfl_xor(st.x, off), __shfl_xor(st.y, off)});
            }
            row_done(jr, best, st);
        }
    }
    __syncthreads();
    if (threadIdx.x >= 64 || a.finish == FINISH_NONE) return;
    // the decision: one wavefront, a lane per row (k <= 64)
    const int j = lane;
    if (a.finish == FINISH_DRAFT) {
        if (j >= 1 && j < k) a.draft_out[(size_t)b * (k - 1) + j - 1] = am[j];
    } else if (denoise) {
        const bool masked = j >= 1 && j < k && in_s[j] == a.mask_id;
        const float c = masked ? cf[j] : 0.f;
        const unsigned long long left = __ballot(masked), above = __ballot(masked && c > a.threshold);
        int top = -1;   // first of the most confident
        float c_top = 0.f;
        for (unsigned long long w = above ? 0ull : left; w; w &= w - 1) {
            const int i = __ffsll((long long)w) - 1;
            const float ci = __shfl(c, i);
            if (top < 0 || ci > c_top) {
                top = i;
                c_top = ci;
            }
        }
        if (masked && (above ? c > a.threshold : j == top)) a.block[(size_t)b * k + j] = am[j];
        if (j == 0) {
            const int n_mask = __popcll(left), n_commit = above ? __popcll(above) : (n_mask > 0 ? 1 : 0);
            a.n_committed[b] = n_commit;
            a.n_masked[b] = n_mask - n_commit;
        }
    } else {
        const int L = __ffsll((long long)~__ballot(j < k - 1 && in_s[j] == am[j])) - 1;   // at most k - 1
        if (j < k) a.committed[(size_t)b * k + j] = j < L ? in_s[j] : (j == L ? am[j] : -1);
        if (j == 0) {
            a.accept_len[b] = L;
            a.next_anchor[b] = am[L];
            if (a.lengths) advance_length(a, b, L + 1);
        }
    }
}

hipError_t launch_finish(const FinishArgs& a, hipStream_t s) {
    const int threads = a.finish == FINISH_REFRESH ? 64 : 64 * (a.k_blk < 16 ? a.k_blk : 16);
    launch(finish_kernel, dim3(a.batch), dim3(threads), s, a);
    return hipGetLastError();
}

// =====================================================================================
// Quadratic self-speculation (Sec. 3.4, Appendix C).  The block of each sequence is the
// chain [anchor, s_1 .. s_{qk-1}] followed by qk groups of qk masks (k_blk = qk(qk+1)
// rows).  The verifier token v_i of position P + i (i = 1..qk) comes from chain row i-1
// (AR), from mask 1 of group i-1 (diffusion), or from their mixture
// lambda * softmax(AR) + (1 - lambda) * softmax(diffusion).  Acceptance is Mode 3's; the
// next speculative tokens are the argmax of masks 2..qk of group L.
// =====================================================================================
// Workgroup (sequence b and position i, vocabulary chunk ch): the argmax key over the chunk
// of lambda * exp(a_n - A) / SA + (1 - lambda) * exp(d_n - D) / SD (lowest index on ties),
// into ens_keys[(b * quad_k + i) * ens_chunks + ch].  Each thread has eight columns of both
// rows in flight at a time.
__global__ void __launch_bounds__(512) quad_ensemble_kernel(FinishArgs a) {
    __shared__ float2 st_s[2];
    __shared__ unsigned long long key_s[8];
    const int qk = a.quad_k, R = a.k_blk, V = a.vocab;
    const int bi = blockIdx.x, b = bi / qk, i = bi % qk, ch = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    if (wave < 2) {
        const float2 st = row_lse(a, b * R + (wave == 0 ? i : qk + i * qk), lane);
        if (lane == 0) st_s[wave] = st;
    }
    __syncthreads();
    const float2 sa = st_s[0], sd = st_s[1];
    const float ca = a.lambda / sa.y, cd = (1.0f - a.lambda) / sd.y;
    const float* la = a.ens_logits + ((size_t)b * 2 * qk + i) * V;
    const float* ld = a.ens_logits + ((size_t)b * 2 * qk + qk + i) * V;
    const int per = (V + a.ens_chunks - 1) / a.ens_chunks;
    const int n0 = ch * per, n1 = min(V, n0 + per), nt = blockDim.x;
    unsigned long long best = 0ull;
    for (int n = n0 + (int)threadIdx.x; n < n1; n += 8 * nt) {
        float xa[8], xd[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = n + u * nt;
            xa[u] = j < n1 ? la[j] : 0.f;
            xd[u] = j < n1 ? ld[j] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = n + u * nt;
            const float p = ca * expf(xa[u] - sa.x) + cd * expf(xd[u] - sd.x);
            if (j < n1) best = umax64(best, argmax_key(p, (uint32_t)j));
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) best = umax64(best, __shfl_xor(best, off));
    if (lane == 0) key_s[wave] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long k2 = 0ull;
        for (int w = 0; w < nw; ++w) k2 = umax64(k2, key_s[w]);
        a.ens_keys[(size_t)bi * a.ens_chunks + ch] = k2;
    }
}

// One workgroup per sequence: verifier tokens, acceptance, commit, next anchor and the next
// speculative tokens.  draft_out may alias draft_in and next_anchor the anchor the pass read.
__global__ void __launch_bounds__(1024) quad_finish_kernel(FinishArgs a) {
    __shared__ int32_t v_s[64];
    __shared__ int L_s;
    const int b = blockIdx.x, qk = a.quad_k, R = a.k_blk;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
    for (int i = wave; i < qk; i += nw) {
        int32_t v;
        if (a.lambda > 0.0f && a.lambda < 1.0f) {   // the ensemble kernel's per-chunk keys
            unsigned long long best = 0ull;
            for (int c = lane; c < a.ens_chunks; c += 64) best = umax64(best, a.ens_keys[(size_t)(b * qk + i) * a.ens_chunks + c]);
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) best = umax64(best, __shfl_xor(best, off));
            v = argmax_key_index(best);
        } else {
            unsigned long long best[2];
            row_keys(a, b * R + (a.lambda >= 1.0f ? i : qk + i * qk), -1, lane, best);
            v = argmax_key_index(best[0]);
        }
        if (lane == 0) v_s[i] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int32_t* sp = a.draft_in + (size_t)b * (qk - 1);
        int L = 0;
        while (L < qk - 1 && sp[L] == v_s[L]) ++L;
        for (int i = 0; i < qk; ++i) a.committed[(size_t)b * qk + i] = i < L ? sp[i] : (i == L ? v_s[L] : -1);
        a.accept_len[b] = L;
        a.next_anchor[b] = v_s[L];
        if (a.lengths) advance_length(a, b, L + 1);
        L_s = L;
    }
    __syncthreads();
    const int L = L_s;
    for (int r = 2 + wave; r <= qk; r += nw) {
        unsigned long long best[2];
        row_keys(a, b * R + qk + L * qk + r - 1, -1, lane, best);
        if (lane == 0) a.draft_out[(size_t)b * (qk - 1) + r - 2] = argmax_key_index(best[0]);
    }
}

hipError_t launch_quad_ensemble(const FinishArgs& a, hipStream_t s) {
    launch(quad_ensemble_kernel, dim3(a.batch * a.quad_k, a.ens_chunks), dim3(512), s, a);
    return hipGetLastError();
}

hipError_t launch_quad_finish(const FinishArgs& a, hipStream_t s) {
    launch(quad_finish_kernel, dim3(a.batch), dim3(64 * (a.quad_k < 16 ? a.quad_k : 16)), s, a);
    return hipGetLastError();
}

// =====================================================================================
// Weight packing into MFMA B-operand tiles, and a fill kernel.
// =====================================================================================
__global__ void __launch_bounds__(256) pack_kernel(PackArgs p) {
    const size_t total = (size_t)p.n_tiles * p.ksteps * 64;
    for (size_t c = (size_t)blockIdx.x * blockDim.x + threadIdx.x; c < total; c += (size_t)gridDim.x * blockDim.x) {
        const int lane = (int)(c % 64);
        const size_t ts = c / 64;
        const int s = (int)(ts % p.ksteps);
        const int t = (int)(ts / p.ksteps);
        const int col = lane & 15;
        const int kk = 32 * s + 8 * (lane >> 4);
        const uint16_t* row = nullptr;
        if (p.kind == PACK_LINEAR) {
            const int n = 16 * t + col;
            if (n < p.out_dim) row = p.src0 + (size_t)n * p.in_dim;
        } else if (p.kind == PACK_QKV) {
            const int D = p.head_dim, tph = D / 16;
            const int hh = t / tph, u = t % tph;
            const int fi = 8 * u + (col & 7);
            const int n = hh * D + ((col < 8) ? fi : D / 2 + fi);
            if (n < p.rows0) row = p.src0 + (size_t)n * p.in_dim;
            else if (n < p.rows0 + p.rows1) row = p.src1 + (size_t)(n - p.rows0) * p.in_dim;
            else if (n < p.out_dim) row = p.src2 + (size_t)(n - p.rows0 - p.rows1) * p.in_dim;
        } else {
            const int f = 8 * t + (col & 7);
            if (f < p.rows0) row = ((col < 8) ? p.src0 : p.src1) + (size_t)f * p.in_dim;
        }
        uint4 v = {0u, 0u, 0u, 0u};
        if (row && kk < p.in_dim) v = *(const uint4*)(row + kk);
        p.dst[c] = v;
    }
}

hipError_t launch_pack(const PackArgs& a, hipStream_t s) {
    const size_t total = (size_t)a.n_tiles * a.ksteps * 64;
    size_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    launch(pack_kernel, dim3((unsigned)blocks), dim3(256), s, a);
    return hipGetLastError();
}

__global__ void fill_zero_kernel(uint32_t* p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
    const size_t n = bytes / 4;
    size_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks == 0) return hipSuccess;
    launch(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), s, (uint32_t*)p, n);
    return hipGetLastError();
}

__global__ void copy_u32_kernel(const uint32_t* src, uint32_t* dst) {
    if (threadIdx.x == 0) *dst = *src;
}

hipError_t launch_copy_u32(const uint32_t* src, uint32_t* dst, hipStream_t s) {
    launch(copy_u32_kernel, dim3(1), dim3(64), s, src, dst);
    return hipGetLastError();
}

}  // namespace nld

#ifdef NLD_TIMELINE
// copies the phase timestamps (8 x 8192 x 8 uint64) to host memory, or clears them (host == NULL)
extern "C" int nld_timeline_read(void* host, size_t bytes) {
    if (!host) {
        static unsigned long long zero[8 * 8192 * 8];
        return (int)hipMemcpyToSymbol(HIP_SYMBOL(nld::g_timeline), zero, sizeof(zero), 0, hipMemcpyHostToDevice);
    }
    return (int)hipMemcpyFromSymbol(host, HIP_SYMBOL(nld::g_timeline), bytes, 0, hipMemcpyDeviceToHost);
}
#endif
