// Skinny GEMMs of the verify forward: Y[t][n] = sum_k X[t][k] W[n][k] for
// T = sum(l_m + 1) query slots (tens to a few hundred) against weight
// matrices of thousands of rows.  At these shapes the work is bound by
// streaming the weights from HBM once, so the kernels are built around that
// stream:
//   * weights are repacked once (at init) into fragment order: the A operand
//     of v_mfma_f32_16x16x32_bf16 for 16 weight rows x 32 k is one 1 KB block
//     laid out lane by lane (lane l: row l % 16, k 8*(l/16)..+7), and the
//     blocks of a 16-row group follow each other along k, so a wave-wide
//     weight load reads 1 KB (or, for the 32x32 form, two 512-byte runs)
//     contiguously;
//   * two MFMA forms share that layout: 32x32x16 tiles (32 slots per tile,
//     measured 2.1 PFLOP/s against 1.2 for the other; every product runs
//     twice, once per activation plane, so the MFMA rate matters even here)
//     and, for the products of small models, 16x16x32 tiles with smaller
//     workgroups;
//   * the activation chunk X[0:T][k0:k0+KC] is staged in LDS (double
//     buffered) and read by all waves of the workgroup as the B operand;
//     activations come as two bf16 planes (hi, lo = x - hi) that are
//     multiplied separately, which carries them at about 16 significant bits;
//   * a wave owns a fixed set of weight rows and multiplies every slot of its
//     workgroup with them, so a weight byte leaves HBM once per call (from six
//     slot tiles on two waves share the rows, above 256 slots two workgroups of
//     one XCD, the second finding them in its L2);
//   * when there are too few column tiles to fill the GPU the k range is
//     split over S workgroups; partial sums are written to a workspace and a
//     second kernel (or a fused consumer) adds them in split order and
//     applies the epilogue (no device-wide fences, deterministic results);
//   * epilogues: fp32 store, SwiGLU silu(g) * u with gate/up rows interleaved
//     per 16-row group, or the lm_head's softmax statistics.
// The fp32 configuration has a product of its own on the fp32 MFMA.
#include <algorithm>

#include "sdv_device.h"
#include "sdv_internal.h"

namespace sdv {

// Cache policy of the two operand streams (the aux word of the buffer
// loads): weights are read once per pass, so they are fetched nontemporal
// (nt), which measured 6.8 TB/s for the bare weight stream against 6.2 TB/s
// with the default policy; the activation chunks, which every workgroup
// re-reads from L2, take sc0.  Together: gate/up at T = 80 104-109 us
// against 117 us in isolation.
constexpr int kWeightAux = 2;
constexpr int kActAux = 1;

struct GemmP {
    const bf16_t* X;
    const bf16_t* Wp;  // packed weights: [vcols/16][K/32][64 lanes][8]
    int K, KT, T, S, kchunks, tiles;  // KT = K / 32 fragments per 16-row group
    // Work split: a wave unit is the row block one wave multiplies (NSUB
    // 16-row groups, or NS 32-row groups); G units in total.  Each k split
    // has WPS workgroups; workgroup w of a split takes units
    // [w*G/WPS, (w+1)*G/WPS), one per wave, so G need not be a multiple of
    // the waves per workgroup (waves past the range load nothing).
    int G, WPS;
    float* part;     // [S][T][vcols] when S > 1
    int vcols;
    void* out;
    int ldo;
    size_t oplane;  // SwiGLU: elements between the hi and lo output planes
    // RMSNorm applied after the product: when nss is set the input planes
    // hold x * gamma (not normalised) and every output of slot t is scaled
    // by rstd(t) = 1 / sqrt(sum_b nss[t][b] / K + eps), which commutes with
    // the product (one factor per slot row)
    const float* nss;
    int nnb;
    float eps;
    // EPI_LMSTAT: per (slot, workgroup) statistics [T][tiles], the logit of
    // each slot's next draft, that draft per slot (-1: none)
    VStat* lstat;
    float* zd;
    const int32_t* dnext;
    // stream-K (unsplit column-split GEMMs that leave CUs idle): the tiles x
    // kchunks (row tile, chunk) pairs are dealt out in tile-major order as
    // sk_nwg contiguous ranges of equal length, one per workgroup; a piece
    // that does not end its tile leaves its sums in partial slot (tile,
    // piece) of `part` and counts itself in sk_cnt[tile]; the tile's last
    // piece waits for that count, adds the earlier pieces in order and runs
    // the epilogue (sk_nwg = 0: off)
    // the piece waits for at most sk_polls polls of the count
    int sk_nwg, sk_maxp, sk_polls;
    // slot groups (direct-staging form): a workgroup computes the MT slot
    // tiles of one group; with more than one group, `tiles` row tiles make
    // tiles * ng work tiles
    int ng;
    // continued sums: the (row tile, split, chunk) triples of a group dealt out
    // as above to sk_nwg workgroups a group; a work tile is shared by two of
    // them at most, and the second continues the sums of the first from a slot
    // of `part` that begins at float sk_off
    size_t sk_off;
    int* sk_cnt;
    int32_t* flags;  // device error bits (bit 2: a stream-K wait gave up)
};

// Work distribution of a 32x32 product: one work tile per workgroup; stream-K
// with a tile's pieces added up by its last; continued sums.
enum { SK_NONE = 0, SK_WAIT = 1, SK_CONT = 2 };

// stream-K: first pair of workgroup w's range, and the workgroup whose range
// holds pair i
__host__ __device__ __forceinline__ int sk_begin(int w, int total, int nwg) {
    return (int)((long long)w * total / nwg);
}
__host__ __device__ __forceinline__ int sk_owner(int i, int total, int nwg) {
    return (int)(((long long)(i + 1) * nwg - 1) / total);
}
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// lm_head epilogue, the part common to both MFMA forms: the per-wave
// statistics of every slot (staged in LDS as [wave][slot]) are merged over
// the workgroup's waves in wave order, i.e. in increasing vocab rows, and
// leave as one 16-byte record per (workgroup, slot)
template <int NTH, int NW, int NSLOT>
__device__ __forceinline__ void lmstat_merge_waves(const GemmP& p, const VStat* stg, int wgi, int tb = 0) {
    for (int i = threadIdx.x; i < NSLOT && tb + i < p.T; i += NTH) {
        VStat st = stg[i];
#pragma unroll
        for (int w = 1; w < NW; ++w) st = vstat_merge(st, stg[w * NSLOT + i]);
        p.lstat[(size_t)(tb + i) * p.tiles + wgi] = st;
    }
}

// statistics of the n logits one lane holds for one slot (rows in
// increasing order); the draft's logit goes to zd when its row is here
template <int N>
__device__ __forceinline__ VStat lane_stat(const float (&z)[N], const int (&row)[N], int d, float* zd) {
    VStat st = vstat_empty();
#pragma unroll
    for (int e = 0; e < N; ++e) {
        if (z[e] > st.v) { st.v = z[e]; st.i = row[e]; }
        if (row[e] == d) *zd = z[e];
    }
    st.m = st.v;
    if (st.m != -INFINITY) {
        float sum = 0.f;
#pragma unroll
        for (int e = 0; e < N; ++e) sum += expf(z[e] - st.m);
        st.s = sum;
    }
    return st;
}

// block sums of one slot row, all loads issued before the sum (at most
// kNormKMax / kNormBlock blocks)
__device__ __forceinline__ void load_row_ss(const GemmP& p, int t, bool on, float (&v)[kNormKMax / kNormBlock]) {
#pragma unroll
    for (int b = 0; b < kNormKMax / kNormBlock; ++b)
        v[b] = on && b < p.nnb ? p.nss[(size_t)t * p.nnb + b] : 0.f;
}
__device__ __forceinline__ float rstd_of(const GemmP& p, const float (&v)[kNormKMax / kNormBlock]) {
    float ss = 0.f;
#pragma unroll
    for (int b = 0; b < kNormKMax / kNormBlock; ++b) ss += v[b];
    return 1.0f / sqrtf(ss / (float)p.K + p.eps);
}
// the same by a wave whose lanes hold slots t, increasing by lane (all lanes on)
__device__ __forceinline__ float row_rstd(const GemmP& p, int t) {
    if (p.nss == nullptr) return 1.0f;
    float ss = 0.f;
    if (p.nnb <= kNormKMax / kNormBlock) {
        for (int b = 0; b < p.nnb; ++b) ss += p.nss[(size_t)t * p.nnb + b];
    } else {
        // a few-slot product's sums, one per few columns: lanes over the blocks
        // of each slot of the wave (every thread walking them: +14 us a layer at
        // 256 blocks)
        const int last = __shfl(t, 63, 64);
        for (int r = __builtin_amdgcn_readfirstlane(t); r <= last; ++r) {
            const float v = lane_blocks_sum(p.nss + (size_t)r * p.nnb, p.nnb, threadIdx.x & 63);
            if (r == t) ss = v;
        }
    }
    return 1.0f / sqrtf(ss / (float)p.K + p.eps);
}
// block sums that do not fit a thread's registers (the few-slot products
// write one per 16 columns): one wave per slot, lanes over the blocks
template <int NW>
__device__ __forceinline__ void row_factors_by_wave(const GemmP& p, float* rsl, int tb, int nsl) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int sl = wave; sl < nsl && tb + sl < p.T; sl += NW) {
        const float ss = lane_blocks_sum(p.nss + (size_t)(tb + sl) * p.nnb, p.nnb, lane);
        if (lane == 0) rsl[sl] = 1.0f / sqrtf(ss / (float)p.K + p.eps);
    }
}

__device__ __forceinline__ float silu(float g) { return g / (1.0f + expf(-g)); }

__device__ __forceinline__ void epi_store4(const GemmP& p, int t, int col, f32x4 v, float sc) {
    *(f32x4*)((float*)p.out + (size_t)t * p.ldo + col) = v * sc;
}

// SwiGLU output as the next GEMM's activation planes: hi = bf16(a) at out,
// lo = bf16(a - hi) one plane (oplane elements) further
__device__ __forceinline__ void swiglu_store4(const GemmP& p, int t, int col, f32x4 g, f32x4 u,
                                              float sc) {
    g *= sc;
    u *= sc;
    bf16_t* o = (bf16_t*)p.out + (size_t)t * p.ldo + col;
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float a = silu(g[e]) * u[e];
        hi[e] = f32_to_bf16(a);
        lo[e] = f32_to_bf16(a - bf16_to_f32((bf16_t)hi[e]));
    }
    *(uint2*)o = uint2{hi[0] | (hi[1] << 16), hi[2] | (hi[3] << 16)};
    *(uint2*)(o + p.oplane) = uint2{lo[0] | (lo[1] << 16), lo[2] | (lo[3] << 16)};
}

// Split-K partial sums of the 32x32 form leave through LDS: the
// workgroup's waves hold consecutive weight rows for every slot, staged as
// [slot][row] (row stride ldr floats), so that each 64-lane store writes
// 1 KB of one partial-sum row instead of 32-byte pieces of 32 rows.  Writes
// nsl slot rows starting at slot t0; only the first nrow rows are the
// workgroup's.  (Kernel traces on one machine at 80 slots: QKV / O / down
// 31.0 / 25.0 / 55.9 -> 29.8 / 23.7 / 53.5 us.)
template <int NTH, int WR>
__device__ __forceinline__ void store_partial_rows(const GemmP& p, const float* stg, int ldr, int split,
                                                   int t0, int nsl, int col0, int nrow) {
    constexpr int P4 = WR / 4;  // 16-byte pieces per staged slot row
    float* base = p.part + ((size_t)split * p.T + t0) * p.vcols + col0;
    for (int i = threadIdx.x; i < nsl * P4; i += NTH) {
        const int sl = i / P4, c4 = (i % P4) * 4;
        if (c4 < nrow) *(f32x4*)(base + (size_t)sl * p.vcols + c4) = *(const f32x4*)(stg + sl * ldr + c4);
    }
}

// 16x16x32 form.  MT: 16-slot tiles.  Staged rows are padded to a stride of an
// odd multiple of 32 bytes: the B-fragment reads of 32 lanes (16 rows at two k
// offsets) then hit distinct banks of the 128-bank LDS, and the staging stores
// are ordered so that the rows written together sit 16/R rows apart (R rows
// per 32 lanes), which also spreads them over every bank.
// The SwiGLU product is always split and reduced by its last split: the S
// workgroups of a row tile each take a k range, store their sums and count
// themselves; the one that counts last adds every split's sums in split order
// and runs the epilogue, so no separate reduction kernel is needed.
template <int MT, int EPI, bool SPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2)))
void k_gemm16(GemmP p) {
    constexpr int NW = 4;                // waves per workgroup
    constexpr int NTH = 64 * NW;         // threads per workgroup
    constexpr int NSUB = 2;              // 16-row weight groups per wave (SwiGLU: a gate/up pair)
    constexpr int PL = 2;                // activation planes
    constexpr int PD = 2;                // chunks of prefetch
    constexpr int KC = 64;               // k per chunk
    constexpr bool LA = EPI == EPI_SWIGLU;
    constexpr int ROWS_PER_TILE = 16;
    constexpr int KS = KC / 32;          // MFMA k-steps per chunk
    constexpr int LDX = KC + 16;         // padded LDS row (bf16 elements)
    constexpr int PPR = KC / 8;          // 16-byte pieces per staged row
    constexpr int RPP = 32 / PPR;        // staged rows per 32 lanes
    constexpr int NPP = MT * 16 * PPR;   // pieces per staged plane
    constexpr int NPC = PL * NPP;        // pieces per staged chunk (all planes)
    constexpr int XPT = NPC / NTH;       // X pieces per thread
    constexpr int PLANE = MT * 16 * LDX;  // LDS elements per plane
    static_assert(NPC % NTH == 0, "whole X pieces per thread");
    static_assert(2 * PL * PLANE * 2 <= 160 * 1024, "X staging exceeds LDS");
    static_assert(!LA || !SPLIT, "last-split reduction: no partial planes");
    __shared__ __attribute__((aligned(16))) bf16_t xs[2][PL * PLANE];
    __shared__ float rsl[SPLIT ? 1 : MT * ROWS_PER_TILE];  // per-slot RMSNorm factor
    __shared__ int la_count;  // LA: splits of this tile counted before this one

    // k split of this workgroup (consecutive workgroups take consecutive
    // splits, so with S a divisor of 8 every XCD works on one k range) and
    // its range of wave units
    constexpr bool KSPLIT = SPLIT || LA;
    const int split = KSPLIT ? blockIdx.x % p.S : 0;
    const int wgi = KSPLIT ? blockIdx.x / p.S : blockIdx.x;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lr = lane & 15, lg = lane >> 4;
    const int mt_act = (p.T + 15) >> 4;

    // Buffer resources: one uniform resource per operand, fixed 32-bit
    // per-lane offsets, uniform chunk offsets.  Out-of-range reads return 0
    // (and fetch nothing: a wave without a unit points past the buffer).
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int unit = wgi * p.G / p.WPS + wv;
    const bool has_unit = unit < (wgi + 1) * p.G / p.WPS;
    const uint64_t wbytes = (uint64_t)p.vcols * (uint64_t)p.K * 2u;
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        (void*)p.Wp, (short)0, (int)(wbytes > 0x7fffffffu ? 0x7fffffffu : wbytes), 0x00020000);
    uint32_t woff[NSUB];
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
        const uint32_t vs = (uint32_t)(unit * NSUB + s);  // 16-row group
        woff[s] = has_unit ? vs * (uint32_t)p.KT * 1024u + (uint32_t)lane * 16u : 0x80000000u;
    }
    const __amdgpu_buffer_rsrc_t xres =
        __builtin_amdgcn_make_buffer_rsrc((void*)p.X, (short)0, PL * p.T * p.K * 2, 0x00020000);

    f32x4 acc[NSUB][MT];
#pragma unroll
    for (int s = 0; s < NSUB; ++s)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[s][m] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int c_begin = split * p.kchunks / p.S;
    const int c_end = (split + 1) * p.kchunks / p.S;

    // Register-ring pipeline with prefetch distance PD chunks: while chunk c
    // is multiplied (X from LDS buffer c&1, W from ring set c % NB), X and W
    // of chunk c+PD are requested into ring set (c+PD) % NB, and X(c+1),
    // requested PD-1 chunks earlier, is stored to the other LDS buffer.  The
    // loop is unrolled by NB so that ring indices are compile-time constants
    // (register copies would force waits on loads still in flight), the
    // loads are unconditional (the chunk index is clamped; the last steps
    // re-read a cached chunk) and scheduling barriers keep the order issue
    // loads -> multiply -> store X.  X rows >= T are read as row T-1: they
    // only feed output slots >= T, which are never stored.
    constexpr int NB = PD + 1;
    uint4 xr[NB][XPT];
    bf16x8 wr[NB][KS][NSUB];
    uint32_t xoff[XPT];
    // staging order q -> LDS row (a permutation within each block of 16 rows)
    auto staged_row = [](int q) { return (q & ~15) | ((q % RPP) * (16 / RPP)) | ((q / RPP) % (16 / RPP)); };
#pragma unroll
    for (int i = 0; i < XPT; ++i) {
        const int idx = (int)threadIdx.x + i * NTH;
        const int pl = idx / NPP, pi = idx % NPP;
        const int r = min(staged_row(pi / PPR), p.T - 1), cc = pi % PPR;
        xoff[i] = (((uint32_t)pl * (uint32_t)p.T + (uint32_t)r) * (uint32_t)p.K + (uint32_t)cc * 8u) * 2u;
    }
    auto load_x = [&](uint4 (&x)[XPT], int c) {
        const int so = c * KC * 2;
#pragma unroll
        for (int i = 0; i < XPT; ++i)
            x[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xres, xoff[i], so, kActAux));
    };
    auto store_x = [&](const uint4 (&x)[XPT], int buf) {
#pragma unroll
        for (int i = 0; i < XPT; ++i) {
            const int idx = threadIdx.x + i * NTH;
            const int pl = idx / NPP, pi = idx % NPP;
            *(uint4*)(&xs[buf][pl * PLANE + staged_row(pi / PPR) * LDX + (pi % PPR) * 8]) = x[i];
        }
    };
    auto load_w = [&](bf16x8 (&w)[KS][NSUB], int c) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int s = 0; s < NSUB; ++s)
                w[ks][s] = __builtin_bit_cast(
                    bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wres, woff[s], (c * KS + ks) * 1024, kWeightAux));
    };
    // The X fragments of all slot tiles of a k-step are read before their
    // MFMAs, and every slot tile of the class is computed (tiles past T multiply clamped
    // copies of row T-1 and are never stored): a per-tile branch would
    // serialise LDS latency and MFMAs tile by tile.
    auto compute = [&](int buf, const bf16x8 (&w)[KS][NSUB]) {
        const bf16_t* xb = xs[buf];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bf16x8 xf[PL][MT];
#pragma unroll
            for (int pl = 0; pl < PL; ++pl)
#pragma unroll
                for (int g = 0; g < MT; ++g)
                    xf[pl][g] = *(const bf16x8*)(xb + pl * PLANE + (g * 16 + lr) * LDX + ks * 32 + 8 * lg);
#pragma unroll
            for (int g = 0; g < MT; ++g)
#pragma unroll
                for (int pl = 0; pl < PL; ++pl)
#pragma unroll
                    for (int s = 0; s < NSUB; ++s)
                        acc[s][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][s], xf[pl][g], acc[s][g], 0, 0, 0);
        }
    };

    const int c_last = c_end - 1;
    // RMSNorm row factors of the tile's slots (epilogues that scale by
    // them): loads issued ahead of the pipeline prologue, the factors go to
    // LDS before the first barrier
    constexpr int NSL = MT * ROWS_PER_TILE;
    constexpr int NSPT = SPLIT ? 1 : (NSL + NTH - 1) / NTH;  // slots per thread
    float ssv[NSPT][kNormKMax / kNormBlock];
    if constexpr (!SPLIT) {
#pragma unroll
        for (int i = 0; i < NSPT; ++i) {
            const int sl = threadIdx.x + i * NTH;
            load_row_ss(p, min(sl, p.T - 1), p.nss != nullptr && sl < NSL, ssv[i]);
        }
    }
#pragma unroll
    for (int u = 0; u < PD; ++u) {
        load_x(xr[u], min(c_begin + u, c_last));
        load_w(wr[u], min(c_begin + u, c_last));
    }
    if constexpr (!SPLIT) {
#pragma unroll
        for (int i = 0; i < NSPT; ++i) {
            const int sl = threadIdx.x + i * NTH;
            if (sl < NSL) rsl[sl] = p.nss != nullptr ? rstd_of(p, ssv[i]) : 1.0f;
        }
        if (p.nss != nullptr && p.nnb > kNormKMax / kNormBlock) {
            __syncthreads();
            row_factors_by_wave<NW>(p, rsl, 0, NSL);
        }
    }
    store_x(xr[0], 0);
    __syncthreads();
    for (int c0 = c_begin; c0 < c_end; c0 += NB) {
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            const int c = c0 + u;
            if (c >= c_end) break;
            load_x(xr[(u + PD) % NB], min(c + PD, c_last));
            load_w(wr[(u + PD) % NB], min(c + PD, c_last));
            __builtin_amdgcn_sched_barrier(0);
            compute((c - c_begin) & 1, wr[u]);
            __builtin_amdgcn_sched_barrier(0);
            store_x(xr[(u + 1) % NB], ((c - c_begin) & 1) ^ 1);
            __syncthreads();
        }
    }

    if constexpr (LA) {
        // The tile's splits exchange their sums through memory at system
        // scope (written through, read past the caches), ordered by the
        // count: each split stores into a slot of its own, waits for the
        // stores, passes a barrier and counts; the split that counts last
        // (no waiting anywhere: every split goes on or leaves at once)
        // resets the count and loads the other slots.  Slot layout: piece
        // j = s * MT + m of thread i at j * NTH + i (16 bytes, coalesced).
        constexpr int PER = NSUB * MT;  // 16-byte accumulator pieces per thread
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(p.part + (size_t)wgi * p.S * (size_t)(NTH * PER * 4)), (short)0, p.S * NTH * PER * 16,
            0x00020000);
#pragma unroll
        for (int s = 0; s < NSUB; ++s)
#pragma unroll
            for (int m = 0; m < MT; ++m)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[s][m]), r,
                                                       ((split * PER + s * MT + m) * NTH + (int)threadIdx.x) * 16,
                                                       0, 17);
        wait_vm<0>();
        __syncthreads();
        if (threadIdx.x == 0)
            la_count = __hip_atomic_fetch_add(p.sk_cnt + wgi, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __syncthreads();
        if (la_count < p.S - 1) return;
        // every split has counted: back to zero for the next launch
        if (threadIdx.x == 0) __hip_atomic_store(p.sk_cnt + wgi, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        // all splits' sums in split order (this split's from its registers)
        f32x4 tot[NSUB][MT];
#pragma unroll
        for (int s = 0; s < NSUB; ++s)
#pragma unroll
            for (int m = 0; m < MT; ++m) tot[s][m] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int sp = 0; sp < p.S; ++sp) {
            if (sp == split) {
#pragma unroll
                for (int s = 0; s < NSUB; ++s)
#pragma unroll
                    for (int m = 0; m < MT; ++m) tot[s][m] += acc[s][m];
                continue;
            }
            u32x4 v[NSUB][MT];
#pragma unroll
            for (int s = 0; s < NSUB; ++s)
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    v[s][m] = __builtin_amdgcn_raw_buffer_load_b128(
                        r, ((sp * PER + s * MT + m) * NTH + (int)threadIdx.x) * 16, 0, 17);
#pragma unroll
            for (int s = 0; s < NSUB; ++s)
#pragma unroll
                for (int m = 0; m < MT; ++m) tot[s][m] += __builtin_bit_cast(f32x4, v[s][m]);
        }
#pragma unroll
        for (int s = 0; s < NSUB; ++s)
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[s][m] = tot[s][m];
    }

    if constexpr (EPI == EPI_LMSTAT) {
        // lane holds D[n = 4*lg + r][t = lr]: a slot's 16 rows of a group sit
        // in lanes lr, lr + 16, lr + 32, lr + 48
        static_assert(!SPLIT, "the lm_head statistics need whole k sums");
        constexpr int NSLOT = MT * 16;
        static_assert(NW * NSLOT * (int)sizeof(VStat) <= (int)sizeof(xs), "statistics staging exceeds LDS");
        VStat* stg = reinterpret_cast<VStat*>(&xs[0][0]);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int t = m * 16 + lr;
            VStat st = vstat_empty();
            if (has_unit && m < mt_act && t < p.T) {
                const float sc = rsl[t];
                float z[NSUB * 4];
                int row[NSUB * 4];
#pragma unroll
                for (int s = 0; s < NSUB; ++s) {
                    const int r0 = (unit * NSUB + s) * 16 + 4 * lg;
                    f32x4 v = acc[s][m] * sc;
                    if (p.out) *(f32x4*)((float*)p.out + (size_t)t * p.ldo + r0) = v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        z[s * 4 + e] = v[e];
                        row[s * 4 + e] = r0 + e;
                    }
                }
                st = lane_stat(z, row, p.dnext[t], p.zd + t);
            }
            st = vstat_merge(st, vstat_shfl_xor(st, 16));
            st = vstat_merge(st, vstat_shfl_xor(st, 32));
            if (lg == 0) stg[wv * NSLOT + t] = st;
        }
        __syncthreads();
        lmstat_merge_waves<NTH, NW, NSLOT>(p, stg, wgi);
        return;
    }
    // lane holds D[n = 4*lg + r][t = lr] of each (sub-tile, slot tile)
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int t = m * 16 + lr;
        if (!(has_unit && m < mt_act && t < p.T)) continue;
        const float sc = SPLIT ? 1.0f : rsl[t];
        if (SPLIT) {
#pragma unroll
            for (int s = 0; s < NSUB; ++s) {
                const int v = (unit * NSUB + s) * 16 + 4 * lg;
                *(f32x4*)(p.part + ((size_t)split * p.T + t) * p.vcols + v) = acc[s][m];
            }
        } else if (EPI == EPI_SWIGLU) {
            // groups 2j / 2j+1 hold gate / up rows 16j..16j+15
#pragma unroll
            for (int s = 0; s < NSUB; s += 2)
                swiglu_store4(p, t, (unit * NSUB + s) / 2 * 16 + 4 * lg, acc[s][m], acc[s + 1][m], sc);
        } else {
#pragma unroll
            for (int s = 0; s < NSUB; ++s)
                epi_store4(p, t, (unit * NSUB + s) * 16 + 4 * lg, acc[s][m], sc);
        }
    }
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// Direct-staging form: the B fragments of N consecutive slot tiles (4 KB
// apart) requested from LDS without a wait, and the wait that leaves at most
// LEFT later requests in flight; the waits take the fragments as operands, so
// nothing that uses them is scheduled before.
template <int N>
__device__ __forceinline__ void lds_read_tiles(bf16x8 (&f)[N], uint32_t a) {
    if constexpr (N == 1) asm volatile("ds_read_b128 %0, %1" : "=&v"(f[0]) : "v"(a) : "memory");
    if constexpr (N == 2)
        asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:4096"
                     : "=&v"(f[0]), "=&v"(f[1]) : "v"(a) : "memory");
    if constexpr (N == 3)
        asm volatile("ds_read_b128 %0, %3\n\tds_read_b128 %1, %3 offset:4096\n\tds_read_b128 %2, %3 offset:8192"
                     : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]) : "v"(a) : "memory");
    static_assert(N >= 1 && N <= 5, "tiles per wave");
    if constexpr (N == 4)
        asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:4096\n\tds_read_b128 %2, %4 offset:8192\n\t"
                     "ds_read_b128 %3, %4 offset:12288"
                     : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]) : "v"(a) : "memory");
    if constexpr (N == 5)
        asm volatile("ds_read_b128 %0, %5\n\tds_read_b128 %1, %5 offset:4096\n\tds_read_b128 %2, %5 offset:8192\n\t"
                     "ds_read_b128 %3, %5 offset:12288\n\tds_read_b128 %4, %5 offset:16384"
                     : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]) : "v"(a) : "memory");
}
template <int LEFT, int N>
__device__ __forceinline__ void lds_wait_tiles(bf16x8 (&f)[N]) {
    if constexpr (N == 1) asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(f[0]) : "n"(LEFT));
    if constexpr (N == 2) asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(f[0]), "+v"(f[1]) : "n"(LEFT));
    if constexpr (N == 3) asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]) : "n"(LEFT));
    if constexpr (N == 4)
        asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]) : "n"(LEFT));
    if constexpr (N == 5)
        asm volatile("s_waitcnt lgkmcnt(%5)"
                     : "+v"(f[0]), "+v"(f[1]), "+v"(f[2]), "+v"(f[3]), "+v"(f[4]) : "n"(LEFT));
}

// 32x32x16 form.  MT: 32-slot tiles of a workgroup; a wave multiplies 64
// weight rows (two 32-row groups), so every B fragment read from LDS feeds two
// MFMAs: four SIMDs issuing 32-cycle MFMAs then ask for 64 bytes per clock of
// LDS reads instead of 128.
// CS = 1, four waves (up to five tiles, one set of accumulators per wave; up
// to four tiles two workgroups share a CU); CS = 2 (column split), eight
// waves: two waves share one row unit and each multiplies MT/2 of the tiles.
// Both hold 256 weight rows per workgroup.
// Slot groups (ng > 1): workgroups b and b + 8 (the same XCD, dispatched
// together) compute the same weight rows for consecutive groups of MT tiles,
// so the second finds the weights in its XCD's L2.
// SK: work distribution.  SK_WAIT, stream-K of an unsplit product (GemmP).
// SK_CONT, for more work tiles than workgroups: each takes an equal run of
// (work tile, chunk) pairs, so at most two share a tile.  It first computes
// the head of its last tile and leaves the sums in memory, then its whole
// tiles, then the tail of its first tile, whose head the workgroup before it
// has left in the meantime: the accumulators start from those sums, and every
// output is one chain of products in order of k, bit for bit that of one
// workgroup per tile.  Nothing waits: both count themselves once, and a tail
// that counts before its head (or whose sk_polls is zero) computes the whole
// tile itself.  Qwen3-32B shapes at T = 359, us: gate/up 321 (adding up the
// pieces of a tile instead: 372), QKV / O / down on average 114.
template <int MT, int EPI, bool SPLIT, int NW, int CS, int SK = SK_NONE>
__global__ __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(1, CS == 2 ? 2 : MT >= 5 ? 1 : MT >= 3 ? 2 : 4)))
void k_gemm32(GemmP p) {
    constexpr int PL = 2;                // activation planes
    constexpr int NS = 2;                // 32-row groups per wave
    constexpr int KC = 64;               // k per chunk
    static_assert(MT % CS == 0 && NW == 4 * CS, "whole tiles per wave, 256 weight rows per workgroup");
    static_assert(SK != SK_WAIT || (!SPLIT && EPI == EPI_SWIGLU), "stream-K: the unsplit SwiGLU product");
    static_assert(SK != SK_CONT || SPLIT || EPI == EPI_SWIGLU, "continued sums: split products and SwiGLU");
    constexpr int MTW = MT / CS;         // slot tiles per wave
    constexpr int NTH = 64 * NW;         // threads per workgroup
    constexpr int PER4 = NS * MTW * 4;   // 16-byte accumulator pieces per thread
    constexpr int KS = KC / 16;          // MFMA k-steps per chunk
    // weight register sets: two, except where the registers hold only one
    constexpr int WD = MT == 8 ? 1 : 2;
    // two X buffers of XBUF elements; the split epilogue stages its partial
    // sums in the same memory, which may need more
    constexpr int XBUF = PL * MT * 32 * KC;
    constexpr int STG_BYTES = SPLIT ? CS * 32 * (NW / CS * NS * 32 + 4) * 4 : EPI == EPI_LMSTAT ? NW / CS * MT * 32 * 16 : 0;
    constexpr int XS_ELEMS = 4 * XBUF >= STG_BYTES ? 2 * XBUF : STG_BYTES / 2;
    static_assert(XS_ELEMS * 2 <= 160 * 1024, "staging exceeds LDS");
    __shared__ __attribute__((aligned(16))) bf16_t xs[XS_ELEMS];
    __shared__ float rsl[SPLIT ? 1 : MT * 32];  // per-slot RMSNorm factor
    __shared__ int sk_seen;  // SK_CONT: count of the shared tile before this workgroup's

    // Work tile of this workgroup: (row tile, k split), for one slot group.
    int bid = blockIdx.x, grp = 0;
    if (SK != SK_WAIT && p.ng > 1) {
        grp = (bid >> 3) % p.ng;
        bid = (bid >> 3) / p.ng * 8 + (bid & 7);
        if (SK == SK_NONE && bid >= p.tiles * p.S) return;  // the grid is rounded up to 8 workgroups per group
    }
    // Stream-K and continued sums: the workgroup's range of (work tile, chunk)
    // pairs is cut at the tile ends into pieces.  The piece of the last tile is
    // taken first (when it does not end its tile, another workgroup needs it).
    // Stream-K then goes on in order, continued sums leave the first tile for
    // the end.  Otherwise one piece: the whole k range of a split.
    const int uch = SK == SK_CONT ? p.kchunks / p.S : p.kchunks;  // chunks per work tile
    int sk_np = 1, sk_wb = 0, sk_we = 0, sk_t0 = 0;
    if constexpr (SK != SK_NONE) {
        const int total = p.tiles * (SPLIT ? p.S : 1) * uch;
        sk_wb = sk_begin(bid, total, p.sk_nwg);
        sk_we = sk_begin(bid + 1, total, p.sk_nwg);
        sk_t0 = sk_wb / uch;
        sk_np = (sk_we - 1) / uch - sk_t0 + 1;
    }
    for (int piece = 0; piece < sk_np; ++piece) {
    // What depends on the thread is computed anew for every piece: kept over the
    // pieces it spills (stream-K 76 -> 32 bytes a lane, gate/up at 231 slots
    // 216.4 -> 214.6 us)
    int tid = threadIdx.x;
    if (SK != SK_NONE) asm volatile("" : "+v"(tid));
    const int wave = tid >> 6, lane = tid & 63;
    const int lc = lane & 31, lh = lane >> 5;
    // the last piece's epilogue reads the row factors this one overwrites
    if (SK != SK_NONE && piece > 0) __syncthreads();
    const int skt = SK == SK_NONE ? 0
                    : sk_t0 + (piece == 0                             ? sk_np - 1
                               : SK == SK_WAIT                        ? piece - 1
                               : piece == sk_np - 1                   ? 0
                                                                      : piece);
    const int wt = SK == SK_NONE ? bid : skt;  // work tile (row tile, split)
    const int split = SPLIT ? wt % p.S : 0;
    const int wgi = SPLIT ? wt / p.S : wt;
    const int tb = grp * MT * 32;  // first slot of the group

    // Buffer resources: one uniform resource per operand, fixed 32-bit
    // per-lane offsets, uniform chunk offsets.  Out-of-range reads return 0
    // (and fetch nothing: a wave without a unit points past the buffer).
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int half = CS == 1 ? 0 : wv % CS;   // which MT/CS slot tiles
    const int wrow = wv / CS;                 // row unit within the workgroup
    const int m0 = half * MTW;
    const int unit = wgi * p.G / p.WPS + wrow;
    const bool has_unit = unit < (wgi + 1) * p.G / p.WPS;
    const uint64_t wbytes = (uint64_t)p.vcols * (uint64_t)p.K * 2u;
    const int wrec = (int)(wbytes > 0x7fffffffu ? 0x7fffffffu : wbytes), xrec = PL * p.T * p.K * 2;
    // The A operand of a 16-k step (lane l: row l % 32, k 8*(l/32)..+7)
    // taken from the 16-row fragments: rows 0-15 / 16-31 are 16-row groups
    // 2g / 2g+1; k-step j sits in fragment j/2 at k 16*(j%2), i.e. lane slot
    // (l % 16) + 16*(l/32) + 32*(j%2).  Per lane that is a fixed offset plus
    // a uniform 512*j.
    uint32_t woff[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const uint32_t g16 = (uint32_t)((unit * NS + s) * 2 + (lc >> 4));
        woff[s] = has_unit ? g16 * (uint32_t)p.KT * 1024u + (uint32_t)((lane & 15) + 16 * lh) * 16u
                           : 0x80000000u;
    }

    f32x16 acc[NS][MTW];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int m = 0; m < MTW; ++m)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[s][m][e] = 0.f;

    // chunks of the work tile that this piece computes
    const int c_split = split * p.kchunks / p.S;
    int c_lo = SK == SK_NONE ? 0 : max(sk_wb - skt * uch, 0);
    const int c_hi = SK == SK_NONE ? (split + 1) * p.kchunks / p.S - c_split : min(sk_we - skt * uch, uch);
    // sums of a shared tile: element j of thread i at j * NTH + i (16-byte
    // pieces, coalesced)
    auto sk_slot = [&](size_t i) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)(p.part + p.sk_off + i * (size_t)(NTH * PER4 * 4)), (short)0,
                                                 NTH * PER4 * 16, 0x00020000);
    };
    if constexpr (SK == SK_CONT) {
        if (c_lo > 0) {
            const int head = (bid - 1) * p.ng + grp;
            if (threadIdx.x == 0) {
                const int n = __hip_atomic_fetch_add(p.sk_cnt + head, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                // the head has counted: back to zero for the next launch
                if (n == 1) __hip_atomic_store(p.sk_cnt + head, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                sk_seen = p.sk_polls > 0 ? n : 0;
            }
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(sk_seen) == 1) {
                const __amdgpu_buffer_rsrc_t r = sk_slot(head);
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int m = 0; m < MTW; ++m)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const f32x4 f = __builtin_bit_cast(
                                f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                           r, (((s * MTW + m) * 4 + q) * NTH + (int)threadIdx.x) * 16, 0, 17));
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[s][m][4 * q + e] = f[e];
                        }
                // (here, so that no wait for them is left to the first products)
                wait_vm<0>();
                __builtin_amdgcn_sched_barrier(0);
            } else {
                c_lo = 0;
            }
        }
    }
    const int c_begin = c_split + c_lo, c_end = c_split + c_hi;
    // RMSNorm row factors of the tile's slots (epilogues that scale by
    // them): loads issued ahead of the pipeline prologue, the factors go to
    // LDS before the first barrier
    constexpr int NSL = MT * 32;
    constexpr int NSPT = SPLIT ? 1 : (NSL + NTH - 1) / NTH;  // slots per thread
    float ssv[NSPT][kNormKMax / kNormBlock];
    if constexpr (!SPLIT) {
#pragma unroll
        for (int i = 0; i < NSPT; ++i) {
            const int sl = threadIdx.x + i * NTH;
            load_row_ss(p, min(tb + sl, p.T - 1), p.nss != nullptr && sl < NSL, ssv[i]);
        }
    }
    // Packed last tile (when the last tile holds at most 16 slots): its rows
    // 0-15 hold their hi plane and rows 16-31 their lo plane, one tile-plane
    // instead of two; the wave that holds it multiplies it in the plane-0
    // phases only.  Not with slot groups, where every slot's sums are one chain
    // (359 slots: 1% of the products' time)
    const int last_n = p.T - tb - (MT - 1) * 32;
    const bool pkl = p.ng == 1 && last_n > 0 && last_n <= 16;
    const bool pkl_half = pkl && half == CS - 1;

    // Two X buffers in LDS, WD weight register sets.  Per chunk c: the direct
    // loads of X(c + 1) into the buffer that chunk c - 1 has left are issued
    // first; phases (k-step, plane) follow, the next phase's fragments
    // requested before this phase's NS * MTW MFMAs; after the last plane of a
    // k-step its weight registers are reloaded with the same k-step of chunk
    // c + WD; the wave then waits for its direct loads of chunk c + 1 and the
    // barrier publishes the buffer.  Chunks past the range are requested from
    // an empty buffer resource, so that nothing is fetched (re-reading the
    // last chunk instead cost a tenth of a ten-chunk split's traffic) and the
    // count of loads in flight stays the same for every chunk.  Three or four
    // buffers and register sets measured the same or slower (T = 16: 3446 us
    // a pass of 16 layers with two, 3503 / 3529 with three / four; T = 80:
    // 4843, 4894 / 5025).
    constexpr int NPH = KS * PL;
    // X is staged by direct global-to-LDS loads: a chunk is MT * 8 blocks
    // of 1 KB, block (plane, tile, row group of 8) holding 8 rows of 64 k
    // (128 B each) whose 16-byte pieces are XOR-swizzled by the row
    // (piece q at position q ^ ((row >> 1) & 7), row within the tile), so
    // that the fragment reads of 16 rows hit 16 different bank groups.
    // A wave's direct load fills one block (lane l: row l / 8, position
    // l % 8), so each lane fetches the piece that belongs to its
    // position; each wave loads MT * 8 / NW blocks per chunk.  Slots >= T are
    // read as slot T-1: they only feed outputs that are never stored.
    constexpr int NBK = MT * 8 / NW;
    typedef __attribute__((address_space(3))) void lds_void;
    uint32_t doff[NBK];
#pragma unroll
    for (int i = 0; i < NBK; ++i) {
        const int blk = wv * NBK + i, pl = blk / (MT * 4), mt = (blk >> 2) % MT, rb = blk & 3;
        const int lrow = rb * 8 + (lane >> 3);
        const int pc = (lane & 7) ^ ((lrow >> 1) & 7);
        // packed last tile: rows 0-15 from the hi plane, 16-31 from the lo
        // plane, of the same 16 slots
        const bool pk = pkl && pl == 0 && mt == MT - 1;
        const int spl = pk ? lrow >> 4 : pl;
        const int row = min(tb + mt * 32 + (pk ? lrow & 15 : lrow), p.T - 1);
        doff[i] = (((uint32_t)spl * (uint32_t)p.T + (uint32_t)row) * (uint32_t)p.K + (uint32_t)pc * 8u) * 2u;
    }
    auto dma_x = [&](int c, int buf) {
        const __amdgpu_buffer_rsrc_t xres =
            __builtin_amdgcn_make_buffer_rsrc((void*)p.X, (short)0, c < c_end ? xrec : 0, 0x00020000);
        bf16_t* base = xs + buf * XBUF + wv * NBK * 512;
#pragma unroll
        for (int i = 0; i < NBK; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(xres, (lds_void*)(base + i * 512), 16, (int)doff[i],
                                                     c * KC * 2, 0, kActAux);
    };
    // fragment reads in inline assembly: the compiler cannot tell them from
    // the direct loads into the other buffer and would wait for every
    // load in flight before them; their completion is waited for
    // explicitly, with the fragments as operands
    const uint32_t xs_addr = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) bf16_t*)xs;
    uint32_t loff[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        loff[ks] = (uint32_t)((lc >> 3) * 1024 + (lc & 7) * 128 + (((2 * ks + lh) ^ ((lc >> 1) & 7)) * 16));
    bf16x8 xq[2][MTW];
    auto read_phase = [&](bf16x8 (&xf)[MTW], int buf, int ph) {
        const int ks = ph / PL, pl = ph % PL;
        lds_read_tiles(xf, xs_addr + (uint32_t)(buf * XBUF * 2) + loff[ks] + (uint32_t)((pl * MT + m0) * 4096));
    };
    bf16x8 wr[WD][KS][NS];
    auto load_w_ks = [&](bf16x8 (&w)[NS], int c, int ks) {
        const __amdgpu_buffer_rsrc_t wres =
            __builtin_amdgcn_make_buffer_rsrc((void*)p.Wp, (short)0, c < c_end ? wrec : 0, 0x00020000);
#pragma unroll
        for (int s = 0; s < NS; ++s)
            w[s] = __builtin_bit_cast(
                bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wres, woff[s], (c * KS + ks) * 512, kWeightAux));
    };
    // the wait below counts loads: only arithmetic may move across these barriers
    dma_x(c_begin, 0);
    __builtin_amdgcn_sched_barrier(1);
#pragma unroll
    for (int u = 0; u < WD; ++u)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) load_w_ks(wr[u][ks], c_begin + u, ks);
    __builtin_amdgcn_sched_barrier(1);
    if constexpr (!SPLIT) {
#pragma unroll
        for (int i = 0; i < NSPT; ++i) {
            const int sl = threadIdx.x + i * NTH;
            if (sl < NSL) rsl[sl] = p.nss != nullptr ? rstd_of(p, ssv[i]) : 1.0f;
        }
        if (p.nss != nullptr && p.nnb > kNormKMax / kNormBlock) {
            __syncthreads();
            row_factors_by_wave<NW>(p, rsl, tb, NSL);
        }
    }
    // When a chunk starts its X has landed, and the weight loads issued after
    // those direct loads may be in flight (loads retire in order).
    wait_vm<WD * NS * KS, true>();  // and the row factors
    barrier_nofence();
    read_phase(xq[0], 0, 0);
    for (int c0 = c_begin; c0 < c_end; c0 += 2) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int c = c0 + u;
            if (c >= c_end) break;
            dma_x(c + 1, u ^ 1);
#pragma unroll
            for (int ph = 0; ph < NPH; ++ph) {
                if (ph + 1 < NPH) {
                    read_phase(xq[(ph + 1) & 1], u, ph + 1);
                    lds_wait_tiles<MTW>(xq[ph & 1]);
                } else {
                    lds_wait_tiles<0>(xq[ph & 1]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < MTW; ++m)
#pragma unroll
                    for (int s = 0; s < NS; ++s)
                        if (!(m == MTW - 1 && ph % PL == 1 && pkl_half))  // packed tile: one plane-phase
                            acc[s][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wr[u % WD][ph / PL][s], xq[ph & 1][m],
                                                                                 acc[s][m], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (ph % PL == PL - 1) load_w_ks(wr[u % WD][ph / PL], c + WD, ph / PL);
            }
            wait_vm<NS * KS>();
            barrier_nofence();
            if (c + 1 < c_end) read_phase(xq[0], u ^ 1, 0);
        }
    }

    int sk_ord = 0;  // SK_WAIT: earlier pieces of this tile to add (the tile's last piece)
    // Partial sums travel through memory at system scope (written through,
    // read past the caches), ordered by the count: stores, wait for them,
    // barrier, then the count; the reader reads the count before it loads.
    auto leave_sums = [&](size_t slot, int* cnt) {
        const __amdgpu_buffer_rsrc_t r = sk_slot(slot);
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int m = 0; m < MTW; ++m)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int j = (s * MTW + m) * 4 + q;
                    const f32x4 v = f32x4{acc[s][m][4 * q], acc[s][m][4 * q + 1], acc[s][m][4 * q + 2],
                                          acc[s][m][4 * q + 3]};
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r,
                                                           (j * NTH + (int)threadIdx.x) * 16, 0, 17);
                }
        wait_vm<0>();
        __syncthreads();
        if (threadIdx.x == 0) {
            const int n = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            // the tail came first and does without: back to zero
            if (SK == SK_CONT && n == 1) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    };
    if constexpr (SK == SK_CONT) {
        if (c_hi < uch) {
            leave_sums(bid * p.ng + grp, p.sk_cnt + bid * p.ng + grp);
            continue;
        }
    }
    if constexpr (SK == SK_WAIT) {
        const int total = p.tiles * p.kchunks;
        const int ord = (int)blockIdx.x - sk_owner(skt * p.kchunks, total, p.sk_nwg);
        if (c_end < p.kchunks) {
            leave_sums((size_t)skt * p.sk_maxp + ord, p.sk_cnt + skt);
            continue;
        }
        if (ord > 0) {
            if (threadIdx.x == 0) {
                for (int polls = 0;; ++polls) {
                    if (polls >= p.sk_polls) {
                        atomicOr(p.flags, 4);
                        break;
                    }
                    if (__hip_atomic_load(p.sk_cnt + skt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) >= ord)
                        break;
                    __builtin_amdgcn_s_sleep(2);
                }
                // back to zero once every earlier piece has counted, also
                // after a wait that gave up (the stream runs the next launch
                // only when all of this one's workgroups have ended)
                __hip_atomic_fetch_sub(p.sk_cnt + skt, ord, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
            __syncthreads();
            sk_ord = ord;  // added tile by tile in the epilogue (fewer live registers)
        }
    }
    // Packed last tile of the direct-staging form (its wave's tile MTW - 1):
    // the sums of its slot i are those of lanes l and l ^ 16 (i = l % 16),
    // added by v_permlane16_swap; run after the earlier stream-K pieces'
    // sums are in
    auto fold_last = [&]() {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const auto pr = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[s][MTW - 1][e]),
                                                                 __float_as_uint(acc[s][MTW - 1][e]), false, false);
                acc[s][MTW - 1][e] = __uint_as_float(pr[0]) + __uint_as_float(pr[1]);
            }
    };
    // Accumulator layout: lane l holds slot t = 32*m + l % 32 and, in
    // registers 4q..4q+3, weight rows 8q + 4*(l/32) + 0..3 of its group.
    if constexpr (EPI == EPI_LMSTAT) {
        // lane l holds slot 32m + l % 32 and rows 8q + 4(l/32) + 0..3 of its
        // 32-row group: a slot's rows sit in lanes l and l ^ 32
        static_assert(!SPLIT, "the lm_head statistics need whole k sums");
        // (column split: the NW / CS row units each stage every slot once)
        constexpr int NSLOT = MT * 32;
        constexpr int NU = NW / CS;  // row units per workgroup
        static_assert(NU * NSLOT * (int)sizeof(VStat) <= (int)sizeof(xs), "statistics staging exceeds LDS");
        VStat* stg = reinterpret_cast<VStat*>(xs);
        if (pkl_half) fold_last();
#pragma unroll
        for (int m = 0; m < MTW; ++m) {
            const int ts = (m0 + m) * 32 + lc, t = tb + ts;
            VStat st = vstat_empty();
            if (has_unit && t < p.T) {
                const float sc = rsl[ts];
                float z[NS * 16];
                int row[NS * 16];
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int r0 = (unit * NS + s) * 32 + 8 * q + 4 * lh;
                        const f32x4 v = f32x4{acc[s][m][4 * q], acc[s][m][4 * q + 1], acc[s][m][4 * q + 2],
                                              acc[s][m][4 * q + 3]} * sc;
                        if (p.out) *(f32x4*)((float*)p.out + (size_t)t * p.ldo + r0) = v;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            z[s * 16 + 4 * q + e] = v[e];
                            row[s * 16 + 4 * q + e] = r0 + e;
                        }
                    }
                st = lane_stat(z, row, p.dnext[t], p.zd + t);
            }
            st = vstat_merge(st, vstat_shfl_xor(st, 32));
            if (lh == 0) stg[wrow * NSLOT + ts] = st;
        }
        __syncthreads();
        lmstat_merge_waves<NTH, NU, NSLOT>(p, stg, wgi, tb);
        return;
    }
    if constexpr (SPLIT) {
        // slot tiles m0 + m of every column half at a time through the (now
        // idle) staging buffer, staged as [half][slot][row]
        constexpr int WR = NW / CS * NS * 32;  // weight rows of the workgroup
        constexpr int LDR = WR + 4;
        static_assert(CS * 32 * LDR * 4 <= (int)sizeof(xs), "partial staging exceeds the X buffer");
        float* stg = reinterpret_cast<float*>(xs);
        const int u0 = wgi * p.G / p.WPS;
        const int nrow = ((wgi + 1) * p.G / p.WPS - u0) * NS * 32;
        if (pkl_half) fold_last();
#pragma unroll
        for (int m = 0; m < MTW; ++m) {
            if (tb + m * 32 >= p.T) break;  // so are the other halves' tiles m + MTW * h
            if (has_unit) {
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *(f32x4*)(stg + (half * 32 + lc) * LDR + (wrow * NS + s) * 32 + 8 * q + 4 * lh) =
                            f32x4{acc[s][m][4 * q], acc[s][m][4 * q + 1], acc[s][m][4 * q + 2], acc[s][m][4 * q + 3]};
            }
            __syncthreads();
#pragma unroll
            for (int h = 0; h < CS; ++h) {
                const int ft = tb + (h * MTW + m) * 32;  // first slot of the tile
                const int nsl = min(32, p.T - ft);
                if (nsl > 0)
                    store_partial_rows<NTH, WR>(p, stg + h * 32 * LDR, LDR, split, ft, nsl, u0 * NS * 32, nrow);
            }
            __syncthreads();
        }
        continue;
    }
#pragma unroll
    for (int m = 0; m < MTW; ++m) {
        if constexpr (SK == SK_WAIT) {
            // the earlier pieces' sums of this slot tile, in piece order
            for (int o = 0; o < sk_ord; ++o) {
                const __amdgpu_buffer_rsrc_t r = sk_slot((size_t)skt * p.sk_maxp + o);
                u32x4 v[NS][4];
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        v[s][q] = __builtin_amdgcn_raw_buffer_load_b128(
                            r, (((s * MTW + m) * 4 + q) * NTH + (int)threadIdx.x) * 16, 0, 17);
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const f32x4 f = __builtin_bit_cast(f32x4, v[s][q]);
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[s][m][4 * q + e] += f[e];
                    }
            }
        }
        if (m == MTW - 1 && pkl_half) fold_last();
        const int ts = (m0 + m) * 32 + lc, t = tb + ts;
        if (!has_unit || t >= p.T) continue;
        const float sc = rsl[ts];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int rg = unit * NS + s;  // 32-row group
            if (EPI == EPI_SWIGLU) {
                // rows 0-15 of the group are gate rows 16*grp.., 16-31 the
                // matching up rows; both sit in the same lane
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    swiglu_store4(p, t, rg * 16 + 8 * q + 4 * lh,
                                  f32x4{acc[s][m][4 * q], acc[s][m][4 * q + 1], acc[s][m][4 * q + 2], acc[s][m][4 * q + 3]},
                                  f32x4{acc[s][m][4 * q + 8], acc[s][m][4 * q + 9], acc[s][m][4 * q + 10], acc[s][m][4 * q + 11]},
                                  sc);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    epi_store4(p, t, rg * 32 + 8 * q + 4 * lh,
                                    f32x4{acc[s][m][4 * q], acc[s][m][4 * q + 1], acc[s][m][4 * q + 2], acc[s][m][4 * q + 3]},
                                    sc);
            }
        }
    }
    }
}

// ---------------------------------------------------------------------------
// Few slots (at most 16) against a matrix of few 16-row groups: a drafting
// model's decode step.  Such a product is a few MB to a few tens of MB of
// weights, a handful of microseconds of HBM time, and what it takes is the
// number of dependent memory round trips; so a workgroup owns NG whole
// 16-row groups, its waves share the k range and request their whole share
// (U fragments of 1 KB per group and step, two steps in flight) before the
// first product, the B operand comes straight from the activation rows (they
// sit in L2; no staging, no barrier in the loop), and the waves' sums meet in
// LDS, so that the epilogue follows in the same launch: no partial planes, no
// reduction kernel.
//   RAW     one plane of raw sums for k_qkrope_bf16
//   SWIGLU  two groups, gate and up
//   RESID   x += sum, h = x * gamma and one sum of squares per workgroup's columns
// PACK (at most 8 slots): columns 0-7 of the B operand are the slots' hi plane
// and 8-15 their lo plane, one load and one MFMA instead of two.
// Qwen3-1.7B, one slot, us a product with its reduction: QKV 7.4 -> 5.6, O
// 6.1 + 2.8 -> 5.7, gate/up 13.6 + 3.8 -> 11.9, down 6.1 + 2.8 -> 8.7 (whole
// 16-row groups: 10.3); the step 1685 -> 1421.
// HALF: a workgroup takes 8 rows of a group (the other lanes of the A operand
// are zero), twice the workgroups where whole groups leave half the CUs idle.
// ---------------------------------------------------------------------------
enum { FEW_RAW = 0, FEW_SWIGLU = 1, FEW_RESID = 2 };
struct FewP {
    const bf16_t* X;   // [2][T][K]
    const bf16_t* Wp;  // packed, [groups][K/32][64][8]
    int K, KT, T, N;   // N: output columns
    int groups;
    float* out;        // RAW: [T][N]
    bf16_t* act;       // SWIGLU: [2][T][N]
    const float* nss;  // SWIGLU: block sums of squares of the input rows
    int nnb;
    float eps;
    float* x;          // RESID: [T][N], gamma [N], h [2][T][N], ssq [T][workgroups]
    const bf16_t* gamma;
    bf16_t* h;
    float* ssq;
};

template <int NW, int EPI, bool PACK, bool HALF>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4, 4)))
void k_gemm_few(FewP p) {
    static_assert(!HALF || EPI != FEW_SWIGLU, "half groups: one group per workgroup");
    constexpr int ROWS = HALF ? 8 : 16;            // output columns per workgroup
    constexpr int NG = EPI == FEW_SWIGLU ? 2 : 1;  // 16-row groups
    constexpr int PL = PACK ? 1 : 2;               // B operands per fragment
    constexpr int U = NG == 2 && !PACK ? 2 : 4;    // fragments per wave and step
    constexpr int LDG = 64 * 4 + 3 * 16;           // staged group (16 floats between the row quads)
    __shared__ float red[NW][NG * LDG];
    __shared__ float rsl[16];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lr = lane & 15, lg = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int g0 = HALF ? blockIdx.x >> 1 : blockIdx.x * NG;
    const int r0 = HALF ? (blockIdx.x & 1) * 8 : 0;  // first row of the group

    // epilogue inputs, requested ahead of the weights: output (slot te, row
    // r0 + ne) of a group is thread te * ROWS + ne's
    const int te = threadIdx.x / ROWS, ne = threadIdx.x % ROWS;
    const bool mine = te < p.T;
    const int col = blockIdx.x * ROWS + ne;
    uint32_t xin = 0;
    uint16_t gin = 0;
    if constexpr (EPI == FEW_RESID) {
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(p.x, (short)0, p.T * p.N * 4, 0x00020000);
        const __amdgpu_buffer_rsrc_t gr =
            __builtin_amdgcn_make_buffer_rsrc((void*)p.gamma, (short)0, p.N * 2, 0x00020000);
        xin = __builtin_amdgcn_raw_buffer_load_b32(xr, mine ? (te * p.N + col) * 4 : (int)0x80000000u, 0, 0);
        gin = __builtin_amdgcn_raw_buffer_load_b16(gr, col * 2, 0, 0);
    }
    constexpr int SPW = ((PACK ? 8 : 16) + NW - 1) / NW;  // slots per wave
    f32x4 ssv[SPW][2];
    if constexpr (EPI == FEW_SWIGLU) {
#pragma unroll
        for (int i = 0; i < SPW; ++i) row_blocks_load(p.nss, p.T, p.nnb, wv + i * NW, lane, ssv[i]);
    }

    const uint64_t wbytes = (uint64_t)p.groups * (uint64_t)p.KT * 1024u;
    const int wrec = (int)(wbytes > 0x7fffffffu ? 0x7fffffffu : wbytes), xrec = 2 * p.T * p.K * 2;
    uint32_t woff[NG], xoff[PL];
#pragma unroll
    for (int g = 0; g < NG; ++g)
        woff[g] = HALF && (lr & 8) != r0 ? 0x80000000u
                                         : (uint32_t)(g0 + g) * (uint32_t)p.KT * 1024u + (uint32_t)lane * 16u;
#pragma unroll
    for (int pl = 0; pl < PL; ++pl) {
        const int slot = PACK ? lr & 7 : lr, plane = PACK ? lr >> 3 : pl;
        // columns without a slot point past the buffer and read as zero
        xoff[pl] = slot < p.T ? ((uint32_t)(plane * p.T + slot) * (uint32_t)p.K + 8u * (uint32_t)lg) * 2u : 0x80000000u;
    }
    bf16x8 w[2][U][NG], x[2][U][PL];
    // step s of this wave: fragments s * NW * U + wv * U .. + U - 1 (KT is a
    // multiple of U); steps past the end read an empty resource
    auto load = [&](bf16x8 (&ww)[U][NG], bf16x8 (&xx)[U][PL], int s) {
        const int f = (s * NW + wv) * U;
        const bool on = f < p.KT;
        const __amdgpu_buffer_rsrc_t wres =
            __builtin_amdgcn_make_buffer_rsrc((void*)p.Wp, (short)0, on ? wrec : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t xres =
            __builtin_amdgcn_make_buffer_rsrc((void*)p.X, (short)0, on ? xrec : 0, 0x00020000);
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int g = 0; g < NG; ++g)
                ww[u][g] = __builtin_bit_cast(
                    bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wres, woff[g], (f + u) * 1024, kWeightAux));
#pragma unroll
            for (int pl = 0; pl < PL; ++pl)
                xx[u][pl] = __builtin_bit_cast(
                    bf16x8, __builtin_amdgcn_raw_buffer_load_b128(xres, xoff[pl], (f + u) * 64, 0));
        }
    };
    f32x4 acc[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int steps = (p.KT + NW * U - 1) / (NW * U);
    load(w[0], x[0], 0);
    load(w[1], x[1], 1);
    __builtin_amdgcn_sched_barrier(0);
    for (int s0 = 0; s0 < steps; s0 += 2) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int pl = 0; pl < PL; ++pl)
#pragma unroll
                    for (int g = 0; g < NG; ++g)
                        acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[b][u][g], x[b][u][pl], acc[g], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            if (s0 + 2 < steps) load(w[b], x[b], s0 + b + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // lane holds rows 4 * lg + e of column lr
#pragma unroll
    for (int g = 0; g < NG; ++g) *(f32x4*)&red[wave][g * LDG + lane * 4 + lg * 16] = acc[g];
    if constexpr (EPI == FEW_SWIGLU) {
#pragma unroll
        for (int i = 0; i < SPW; ++i) {
            const float ss = row_blocks_sum(ssv[i], p.nnb, lane);
            if (lane == 0 && wv + i * NW < 16) rsl[wv + i * NW] = 1.0f / sqrtf(ss / (float)p.K + p.eps);
        }
    }
    __syncthreads();
    if (threadIdx.x >= 16 * ROWS) return;
    // sums of (slot te, row r0 + ne) in wave order
    float v[NG];
    const int o = te * 4 + ((r0 + ne) >> 2) * 80 + (ne & 3);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        float a = 0.f;
#pragma unroll
        for (int q = 0; q < NW; ++q) a += red[q][g * LDG + o];
        if constexpr (PACK) {
            float lo = 0.f;
            if (te < 8) {
#pragma unroll
                for (int q = 0; q < NW; ++q) lo += red[q][g * LDG + o + 32];
            }
            a += lo;
        }
        v[g] = a;
    }
    if constexpr (EPI == FEW_RAW) {
        if (mine) p.out[(size_t)te * p.N + col] = v[0];
    } else if constexpr (EPI == FEW_SWIGLU) {
        if (mine) {
            const float sc = rsl[te];
            st_act(p.act, (size_t)p.T * p.N, (size_t)te * p.N + col, silu(v[0] * sc) * (v[1 % NG] * sc));
        }
    } else {
        const float r = __uint_as_float(xin) + v[0];
        if (mine) {
            p.x[(size_t)te * p.N + col] = r;
            st_act(p.h, (size_t)p.T * p.N, (size_t)te * p.N + col, r * bf16_to_f32(gin));
        }
        float ss = r * r;
#pragma unroll
        for (int d = ROWS / 2; d > 0; d >>= 1) ss += __shfl_xor(ss, d, ROWS);
        if (mine && ne == 0) p.ssq[(size_t)te * (p.N / ROWS) + blockIdx.x] = ss;
    }
}

// Sum of the S split-K partials (in split order) plus the epilogue; one
// thread per 4 output columns of one slot.
template <int EPI>
__global__ __launch_bounds__(256) void k_splitk_reduce(GemmP p) {
    const int ncols = EPI == EPI_SWIGLU ? p.vcols / 2 : p.vcols;
    const int per_row = ncols / 4;
    const int all = p.T * per_row, idx = min((int)(blockIdx.x * 256 + threadIdx.x), all - 1);
    const int t = idx / per_row, c = (idx % per_row) * 4;
    const float sc = row_rstd(p, t);
    if ((int)(blockIdx.x * 256 + threadIdx.x) >= all) return;
    const size_t stride = (size_t)p.T * p.vcols;
    const float* base = p.part + (size_t)t * p.vcols;
    if (EPI == EPI_SWIGLU) {
        const int vg = (c / 16) * 32 + (c % 16);  // gate group 2j, up group 2j+1
        f32x4 g = f32x4{0.f, 0.f, 0.f, 0.f}, u = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < p.S; ++s) {
            g += *(const f32x4*)(base + s * stride + vg);
            u += *(const f32x4*)(base + s * stride + vg + 16);
        }
        swiglu_store4(p, t, c, g, u, sc);
    } else {
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < p.S; ++s) v += *(const f32x4*)(base + s * stride + c);
        epi_store4(p, t, c, v, sc);
    }
}

// Weight repack into fragment order.  One wave per (16-row group, 32-k step)
// fragment; lane (r, g) = (lane % 16, lane / 16) copies row r, k 8g..8g+7.
// mode 0: virtual rows are the concatenation of up to three row-major
// segments (QKV); mode 1: groups 2j / 2j+1 are rows 16j.. of src0 / src1
// (SwiGLU gate / up).
__global__ __launch_bounds__(256) void k_pack(const bf16_t* src0, const bf16_t* src1,
                                              const bf16_t* src2, int seg1, int seg2, int mode,
                                              int K, int groups, bf16_t* dst) {
    const int KT = K / 32;
    const long long f = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (f >= (long long)groups * KT) return;
    const int lane = threadIdx.x & 63;
    const int vs = (int)(f / KT), ks = (int)(f % KT);
    const int r = lane & 15, g = lane >> 4;
    const bf16_t* row;
    if (mode == 1) {
        row = ((vs & 1) ? src1 : src0) + (size_t)((vs >> 1) * 16 + r) * K;
    } else {
        const int v = vs * 16 + r;
        row = v < seg1 ? src0 + (size_t)v * K
              : v < seg2 ? src1 + (size_t)(v - seg1) * K : src2 + (size_t)(v - seg2) * K;
    }
    *(uint4*)(dst + ((size_t)f * 64 + lane) * 8) = *(const uint4*)(row + ks * 32 + 8 * g);
}

void launch_pack(const void* s0, const void* s1, const void* s2, int seg1, int seg2, int mode,
                 int K, int vrows, void* dst, hipStream_t s) {
    const long long frags = (long long)(vrows / 16) * (K / 32);
    hipLaunchKernelGGL(k_pack, dim3((unsigned)((frags + 3) / 4)), dim3(256), 0, s,
                       (const bf16_t*)s0, (const bf16_t*)s1, (const bf16_t*)s2, seg1, seg2, mode, K,
                       vrows / 16, (bf16_t*)dst);
}

// ---------------------------------------------------------------------------
// fp32 configuration: v_mfma_f32_16x16x4_f32 (fp32 products and sums).  A
// workgroup computes 16 output columns of 16 slots; its four waves take every
// fourth block of 16 k and their sums are added in wave order through LDS.
// Lane l reads four consecutive k of weight row l % 16 and of slot l % 16 at
// k 4 * (l / 16) of its block, and the block's four MFMAs take element e of
// both, so every row is read in 64-byte pieces; the order of k within a block
// is the same on both sides, which is all the product needs.  Small models
// are bound by latency: short k loops, many workgroups (16 slots, 1024 x 256:
// 35 -> 3.7 us, 1024 x 512 68 -> 4.9 us against one thread per output walking
// its weight row).
// VEC: 16-byte loads (k a multiple of 4, weights and input 16-byte aligned);
// else element by element.  Rows and slots past the end read the last one
// (their outputs are not stored), k past the end reads as zero.
// ---------------------------------------------------------------------------
struct GemmF {
    const float* X;
    const float* W0;
    const float* W1;
    const float* W2;
    int seg1, seg2, N, K, T;
    float* out;
    int ldo;
};

template <bool SWIGLU, bool VEC>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmF p) {
    constexpr int NA = SWIGLU ? 2 : 1;  // weight matrices (SwiGLU: gate and up)
    __shared__ f32x4 part[3][NA][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lr = lane & 15, lg = lane >> 4;
    const int n0 = blockIdx.x * 16, t0 = blockIdx.y * 16;
    const int c = min(n0 + lr, p.N - 1), t = min(t0 + lr, p.T - 1);
    const float* x = p.X + (size_t)t * p.K;
    const float* w[NA];
    if constexpr (SWIGLU) {
        w[0] = p.W0 + (size_t)c * p.K;
        w[1] = p.W1 + (size_t)c * p.K;
    } else {
        w[0] = c < p.seg1 ? p.W0 + (size_t)c * p.K
               : c < p.seg2 ? p.W1 + (size_t)(c - p.seg1) * p.K
                            : p.W2 + (size_t)(c - p.seg2) * p.K;
    }
    auto load4 = [&](const float* r, int k) -> f32x4 {
        if (VEC) return k < p.K ? *(const f32x4*)(r + k) : f32x4{0.f, 0.f, 0.f, 0.f};
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = k + e < p.K ? r[k + e] : 0.f;
        return v;
    };
    f32x4 acc[NA];
#pragma unroll
    for (int a = 0; a < NA; ++a) acc[a] = f32x4{0.f, 0.f, 0.f, 0.f};
    constexpr int UN = 4;  // blocks of this wave in flight
    for (int k0 = wave * 16; k0 < p.K; k0 += 64 * UN) {
        f32x4 xv[UN], wv[NA][UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            xv[u] = load4(x, k0 + 64 * u + 4 * lg);
#pragma unroll
            for (int a = 0; a < NA; ++a) wv[a][u] = load4(w[a], k0 + 64 * u + 4 * lg);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int a = 0; a < NA; ++a)
                    acc[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[a][u][e], xv[u][e], acc[a], 0, 0, 0);
    }
    if (wave > 0) {
#pragma unroll
        for (int a = 0; a < NA; ++a) part[wave - 1][a][lane] = acc[a];
    }
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int a = 0; a < NA; ++a) acc[a] += part[u][a][lane];
    // lane holds columns n0 + 4 * lg + e of slot t0 + lr
    if (t0 + lr >= p.T) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int n = n0 + 4 * lg + e;
        if (n < p.N) p.out[(size_t)(t0 + lr) * p.ldo + n] = SWIGLU ? silu(acc[0][e]) * acc[NA - 1][e] : acc[0][e];
    }
}

// ---------------------------------------------------------------------------
// host-side configuration
// ---------------------------------------------------------------------------

// Tile shape of a product.  F: MFMA form; MT: slot tiles (of 16 or 32 slots)
// of a workgroup; NW: waves; CS: column split; NG: slot groups; KC: k per
// chunk; UR: weight rows of a row unit (one wave's, or CS waves'); FILL:
// split policy, see choose_splits.
struct GemmShape { int F, MT, NW, CS, NG, KC, UR, FILL; };

// The 16x16 form (four-wave workgroups of 128 weight rows, 64-k chunks) serves
// products up to 96 slots that are too small to fill the GPU with 256-row
// workgroups of enough k each; the 32x32 form serves everything else, with
// the tile shape that measured fastest per slot count.  Against the forms it
// replaced (one machine, Qwen3-32B shapes, us): T = 16 gate/up 80.0 -> 79.6,
// lm_head 279 -> 270; T = 60 100 -> 96, 328 -> 308; T = 96 156 -> 125, 470 -> 352,
// the three projections together 129 -> 101 on average of three; T = 128 175 -> 157,
// 534 -> 424; T = 160 202 -> 159; T = 192 229 -> 181; T = 224 275 -> 217; T = 300
// (13-tile four-wave tiles with 16-k chunks before) 650 -> 274; T = 384 715 -> 316.
static GemmShape shape_for(int T, int vcols, bool raw, int K) {
    const bool wide = vcols % 256 == 0;
    constexpr int kT32 = 97;  // slot counts the 16x16 form's tiles end at
    const GemmShape g16{16, (T + 15) / 16, 4, 1, 1, 64, 32, 0};
    if (T < kT32) {
        // split-K partial GEMMs with few weight rows (the Qwen3-1.7B shapes):
        // when 256-row workgroups with at least two 128-k chunks per split
        // cannot fill 90% of the CUs, 128-row ones give twice the workgroups
        // (QKV / O / down at T = 60 8.5-11.2 us against 11.2-17.2 us)
        if (raw && wide) {
            const int tiles8 = vcols / 256;
            const int s8 = std::min(std::max(1, K / 128 / 2), std::max(1, cu_count() / tiles8));
            if (10 * tiles8 * s8 < 9 * cu_count()) return GemmShape{16, g16.MT, 4, 1, 1, 64, 32, 1};
        }
        // SwiGLU products of fewer than a quarter as many 256-row tiles as
        // CUs (the Qwen3-1.7B gate/up: 48): 128-row tiles split to fill the
        // CUs (two splits, 192 workgroups; at T = 60 three splits 26.9, four
        // 24.6, unsplit 28.7, two 23.1 us), reduced by the last split
        // (launch_gemm)
        if (!raw && wide && vcols / 256 * 4 < cu_count()) return GemmShape{16, g16.MT, 4, 1, 1, 64, 32, 1};
        // an lm_head over a short k (the Qwen3-1.7B one: 151936 x 2048,
        // weight-bound at these slot counts): 1187 shorter workgroups leave a
        // shorter tail than 594
        if (!raw && !wide && vcols % 32 == 0 && K <= 2048) return g16;
    }
    const int mt = (T + 31) / 32;
    auto s32 = [](int MT, int CS, int NG) { return GemmShape{32, MT, 4 * CS, CS, NG, 64, 64, 1}; };
    if (mt <= 5) return s32(mt, 1, 1);
    // six tiles and up: the column split is faster than four waves with all
    // tiles (T = 384 in two groups of six, measured with a tile's pieces added
    // up: gate/up 390 against 410 us)
    if (mt == 6) return s32(6, 2, 1);
    if (mt <= 8) return s32(8, 2, 1);
    // two slot groups; five tiles do not halve, so they take four waves
    // (T = 300: gate/up 274 us against 311 for two groups of six)
    if (mt <= 10) return s32(5, 1, 2);
    if (mt <= 12) return s32(6, 2, 2);
    return s32(8, 2, 2);  // three groups of five: 418 against 394 us at T = 400
}

typedef void (*GemmFn)(GemmP);
typedef void (*ReduceFn)(GemmP);

// Activations always come as two planes (hi, lo); split-K kernels write raw
// partial planes and the epilogue runs in the reducer.
template <int MT>
static GemmFn pick16(bool split, int epi) {
    if (split) return k_gemm16<MT, EPI_STORE, true>;
    return epi == EPI_LMSTAT ? k_gemm16<MT, EPI_LMSTAT, false> : k_gemm16<MT, EPI_STORE, false>;
}

template <int MT, int CS>
static GemmFn pick32(bool split, int epi, int sk) {
    if constexpr (MT >= 5)
        if (sk == SK_CONT)
            return split ? k_gemm32<MT, EPI_STORE, true, 4 * CS, CS, SK_CONT>
                         : k_gemm32<MT, EPI_SWIGLU, false, 4 * CS, CS, SK_CONT>;
    if (split) return k_gemm32<MT, EPI_STORE, true, 4 * CS, CS>;
    switch (epi) {
        case EPI_SWIGLU:
            if constexpr (MT == 8)
                if (sk == SK_WAIT) return k_gemm32<MT, EPI_SWIGLU, false, 4 * CS, CS, SK_WAIT>;
            return k_gemm32<MT, EPI_SWIGLU, false, 4 * CS, CS>;
        case EPI_LMSTAT: return k_gemm32<MT, EPI_LMSTAT, false, 4 * CS, CS>;
        default: return k_gemm32<MT, EPI_STORE, false, 4 * CS, CS>;
    }
}

static GemmFn pick(const GemmShape& sh, bool split, int epi, int sk = SK_NONE) {
    if (sh.F == 16) {
        switch (sh.MT) {
            case 1: return pick16<1>(split, epi);
            case 2: return pick16<2>(split, epi);
            case 3: return pick16<3>(split, epi);
            case 4: return pick16<4>(split, epi);
            case 5: return pick16<5>(split, epi);
            default: return pick16<6>(split, epi);
        }
    }
    switch (sh.MT) {
        case 1: return pick32<1, 1>(split, epi, sk);
        case 2: return pick32<2, 1>(split, epi, sk);
        case 3: return pick32<3, 1>(split, epi, sk);
        case 4: return pick32<4, 1>(split, epi, sk);
        case 5: return pick32<5, 1>(split, epi, sk);
        case 6: return pick32<6, 2>(split, epi, sk);
        default: return pick32<8, 2>(split, epi, sk);
    }
}

// the last-split SwiGLU product on the 16x16 tiles (17-96 slots: products this
// small are the few-slot form's up to 16)
static GemmFn pick_la(const GemmShape& sh) {
    if (sh.F != 16) return nullptr;
    switch (sh.MT) {
        case 2: return k_gemm16<2, EPI_SWIGLU, false>;
        case 3: return k_gemm16<3, EPI_SWIGLU, false>;
        case 4: return k_gemm16<4, EPI_SWIGLU, false>;
        case 5: return k_gemm16<5, EPI_SWIGLU, false>;
        case 6: return k_gemm16<6, EPI_SWIGLU, false>;
    }
    return nullptr;
}

static ReduceFn pick_reduce(int epi) {
    switch (epi) {
        case EPI_SWIGLU: return k_splitk_reduce<EPI_SWIGLU>;
        default: return k_splitk_reduce<EPI_STORE>;
    }
}

int cu_count() {  // cached
    static int n = 0;
    if (n == 0) {
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;
    }
    return n;
}

// k splits.  fill: the largest count keeping the grid within one workgroup
// per CU, splits of unequal chunk counts allowed, at least two chunks per
// split (measured on the 32B shapes at T = 80: QKV 40 tiles x 6 = 240
// workgroups 27.2 us vs x 5 30.7 us, O 20 x 12 23.9 vs x 8 27.4, down 20 x 12
// 52.6 vs x 10 57.1; the extra partial sums cost the consumers less than the
// idle CUs cost the GEMM, while twice the splits, two workgroups per CU, cost
// more than they give: 34.8 against 33.8 us on average of the three.  On the
// 1.7B shapes one-chunk splits lose to pipeline start-up and partial-sum
// traffic).  Otherwise (a divisor of kchunks): the largest count giving 1.25
// to 1.75 workgroups per CU, else the smallest giving at least 1.25.
static int choose_splits(int tiles, int kchunks, bool fill) {
    if (fill) {
        const int hi = cu_count();
        if (tiles * 2 > hi) return 1;
        return std::max(1, std::min(std::max(1, kchunks / 2), hi / tiles));
    }
    const int lo = cu_count() * 5 / 4, hi = cu_count() * 7 / 4;
    if (tiles >= lo) return 1;
    int best = 0;
    for (int s = 2; s <= kchunks; ++s)
        if (kchunks % s == 0 && tiles * s >= lo && tiles * s <= hi) best = s;
    if (best) return best;
    for (int s = 2; s <= kchunks; ++s)
        if (kchunks % s == 0 && tiles * s >= lo) return s;
    return kchunks;
}

size_t gemm_partial_floats(const Dims& D, int Tmax) {
    // fp32 path: one plane of the widest raw output
    if (!D.bf16) return (size_t)Tmax * (size_t)std::max(D.nqkv(), D.d);
    // the split count is bounded by the CU count over the tile count, so
    // S * vcols <= ~2 * (CUs * NT) for every call; reserve generously
    // (three planes' worth also holds the stream-K partial slots of the
    // gate/up product at 225-256 slots: 200 tiles x 2 x 65536 floats on the
    // Qwen3-32B shape)
    const size_t widest = (size_t)std::max(std::max(D.nqkv(), D.d), 2 * D.F);
    return (size_t)Tmax * std::max<size_t>(widest * 3, (size_t)65536);
}


// Few-slot products.  PACK needs at most 8 slots; unpacked, an activation
// fragment is twice a weight fragment, so only the gate/up product, which
// shares it between two groups, still reads no more activations than weights.
// (14 slots: gate/up 16.2 -> 15.5 us; the others 8.2-15.6 against 7.5-9.9.)
// The workgroups must all be resident at once (two eight-wave ones or one
// sixteen-wave one per CU): with more (the Qwen3-32B projections) the tiled
// forms' split k is faster (8 slots, 16 layers: 3370 against 3900 us).  Returns
// 0 when another form takes the call, else the columns of a workgroup.
static int try_few(const Dims& D, const GemmCall& g, const SlotBufs& sb, hipStream_t s) {
    const bool swiglu = g.epi == EPI_SWIGLU;
    if (g.T > (swiglu ? 16 : 8) || g.K % 128 || g.N % 16 || g.epi == EPI_LMSTAT) return 0;
    if (swiglu ? g.norm_ss == nullptr || g.norm_nb > kFewBlocks || g.ldo != g.N : !g.raw) return 0;
    int wgs = g.N / 16;
    if (wgs > (swiglu ? 2 : 1) * cu_count()) return 0;
    const bool half = !swiglu && 2 * wgs <= cu_count();
    if (half) wgs *= 2;
    FewP p{};
    p.X = (const bf16_t*)g.X;
    p.Wp = (const bf16_t*)g.Wp;
    p.K = g.K;
    p.KT = g.K / 32;
    p.T = g.T;
    p.N = g.N;
    p.groups = (swiglu ? 2 : 1) * (g.N / 16);
    p.eps = D.eps;
    if (swiglu) {
        p.act = (bf16_t*)g.out;
        p.nss = g.norm_ss;
        p.nnb = g.norm_nb;
        const auto fn = g.T <= 8 ? k_gemm_few<8, FEW_SWIGLU, true, false> : k_gemm_few<8, FEW_SWIGLU, false, false>;
        hipLaunchKernelGGL(fn, dim3(wgs), dim3(512), 0, s, p);
        return 16;
    }
    const bool resid = g.res_gamma && wgs <= kFewBlocks;
    if (resid) {
        p.x = sb.x;
        p.gamma = (const bf16_t*)g.res_gamma;
        p.h = (bf16_t*)sb.h;
        p.ssq = sb.ssq;
    } else {
        if (g.res_gamma) return 0;
        p.out = sb.gpart;
    }
    const auto fn = resid ? (half ? k_gemm_few<16, FEW_RESID, true, true> : k_gemm_few<16, FEW_RESID, true, false>)
                          : (half ? k_gemm_few<16, FEW_RAW, true, true> : k_gemm_few<16, FEW_RAW, true, false>);
    hipLaunchKernelGGL(fn, dim3(wgs), dim3(1024), 0, s, p);
    return half ? 8 : 16;
}

int launch_gemm(const Dims& D, const GemmCall& g, const SlotBufs& sb, hipStream_t s) {
    if (!D.bf16) {
        GemmF p;
        p.X = (const float*)g.X;
        p.W0 = (const float*)g.W[0];
        p.W1 = (const float*)(g.nseg > 1 ? g.W[1] : g.W[0]);
        p.W2 = (const float*)(g.nseg > 2 ? g.W[2] : g.W[0]);
        p.seg1 = g.nseg > 1 ? g.seg[1] : (1 << 30);
        p.seg2 = g.nseg > 2 ? g.seg[2] : (1 << 30);
        p.N = g.N;
        p.K = g.K;
        p.T = g.T;
        p.out = g.raw ? sb.gpart : (float*)g.out;
        p.ldo = g.raw ? g.N : g.ldo;
        const bool swiglu = !g.raw && g.epi == EPI_SWIGLU;
        const bool vec = g.K % 4 == 0 &&
                         (((uintptr_t)p.X | (uintptr_t)p.W0 | (uintptr_t)p.W1 | (uintptr_t)p.W2) & 15) == 0;
        const auto fn = swiglu ? (vec ? k_gemm_f32<true, true> : k_gemm_f32<true, false>)
                               : (vec ? k_gemm_f32<false, true> : k_gemm_f32<false, false>);
        hipLaunchKernelGGL(fn, dim3((g.N + 15) / 16, (g.T + 15) / 16), dim3(256), 0, s, p);
        return 1;
    }
    if (const int cols = try_few(D, g, sb, s)) return g.res_gamma ? -cols : 1;
    const int vcols = g.epi == EPI_SWIGLU ? 2 * g.N : g.N;
    const GemmShape sh = shape_for(g.T, vcols, g.raw != 0, g.K);
    GemmP p;
    p.X = (const bf16_t*)g.X;
    p.Wp = (const bf16_t*)g.Wp;
    p.K = g.K;
    p.KT = g.K / 32;
    p.T = g.T;
    p.kchunks = g.K / sh.KC;
    p.vcols = vcols;
    // workgroups of NW waves; a last partial workgroup when the row count is
    // not a multiple of NW units (its surplus waves load and store nothing)
    const int units = p.vcols / sh.UR;
    const int upw = sh.NW / sh.CS;  // row units per workgroup
    p.tiles = (units + upw - 1) / upw;
    int S = g.epi == EPI_LMSTAT ? 1 : choose_splits(p.tiles * sh.NG, p.kchunks, sh.FILL);
    // Two slot groups over a long k: the splits of 128-row workgroups at 1.25 to
    // 1.75 a CU (Qwen3-32B QKV / O / down: 5 / 8 / 10 where a grid within the
    // CUs has 3 / 6 / 6).  The sums are then added in the same order as by the
    // plain 128-row form, which close decisions depend on; and the workgroups
    // continue each other's sums, so that the count need not fit the CUs.
    if (sh.NG > 1 && g.epi != EPI_LMSTAT) {
        const int s128 = choose_splits((vcols + 127) / 128, p.kchunks, false);
        if (p.kchunks % s128 == 0 && p.kchunks / s128 >= 16) S = s128;
    }
    // four-wave split-K tiles over a short k (the Qwen3-1.7B QKV and O
    // projections, k = 2048): half the splits, so each split keeps four
    // 64-k chunks and the consumer reads half the partial planes (one
    // machine at T = 60, each with its consumer: QKV 18.8 -> 18.4 us, O
    // 14.3 -> 14.0 us per layer; the down projection, k = 6144, is slower
    // so: 19.4 -> 20.0 us)
    if (g.raw && sh.F == 16 && sh.FILL && g.K <= 2048) S = std::max(1, S / 2);
    // (the 16x16 SwiGLU form is a split one; its row tiles are fewer than half
    // the CUs and k at least four chunks, so that there are two anyway)
    if (sh.F == 16 && g.epi == EPI_SWIGLU) S = std::max(S, 2);
    while (S > 1 && (size_t)S * g.T * p.vcols > sb.gpart_floats) {
        int t = S - 1;
        while (t > 1 && p.kchunks % t) --t;
        S = t;
    }
    p.S = S;
    p.G = units;
    p.WPS = p.tiles;
    p.part = sb.gpart;
    p.out = g.out;
    p.ldo = g.ldo;
    p.oplane = (size_t)g.T * g.ldo;  // SwiGLU output planes are [2][T][ldo]
    p.nss = g.norm_ss;
    p.nnb = g.norm_nb;
    p.eps = D.eps;
    p.lstat = reinterpret_cast<VStat*>(g.lstat);
    p.zd = g.zd;
    p.dnext = g.dnext;
    if (g.groups_out) *g.groups_out = p.tiles;
    // Stream-K for an unsplit SwiGLU product of fewer row tiles than CUs (the
    // Qwen3-32B gate/up: 200) at 225-256 slots, where the idle CUs cost most.
    // Its last pieces wait for earlier workgroups, so it stays out where it
    // gives little: 16 layers at T = 132 / 160 / 192 / 224 took 6545 / 6804 /
    // 7527 / 9111 us with it, 6640 / 6841 / 7584 / 9260 take without (the
    // weights' stream bounds the smaller ones).
    p.sk_nwg = 0;
    p.sk_maxp = 0;
    p.sk_off = 0;
    p.ng = sh.NG;
    p.sk_polls = g.sk_polls;
    p.sk_cnt = g.sk_cnt;
    p.flags = g.flags;
    if (!g.raw && g.epi == EPI_SWIGLU && sh.F == 32 && sh.MT == 8 && sh.NG == 1 && g.T > 224 && S == 1 &&
        g.sk_cnt && g.flags && p.tiles < cu_count() && p.tiles <= kSkCounters) {
        const int total = p.tiles * p.kchunks, nwg = std::min(cu_count(), total);
        int maxp = 0;  // most pieces of a tile before its last
        for (int t = 0; t < p.tiles; ++t)
            maxp = std::max(maxp, sk_owner(t * p.kchunks + p.kchunks - 1, total, nwg) -
                                      sk_owner(t * p.kchunks, total, nwg));
        const size_t slot_floats = (size_t)256 * 8 * 32;  // 256 rows, eight tiles of 32 slots
        if (maxp >= 1 && (size_t)p.tiles * maxp * slot_floats <= sb.gpart_floats) {
            p.sk_nwg = nwg;
            p.sk_maxp = maxp;
            hipLaunchKernelGGL(pick(sh, false, g.epi, SK_WAIT), dim3(nwg), dim3(64 * sh.NW), 0, s, p);
            return 1;
        }
    }
    // Continued sums for two slot groups whose work tiles are more than the
    // CUs and no whole multiple
    int sk = SK_NONE;
    const bool split = g.raw || S > 1;
    const int per_group = cu_count() / (8 * p.ng) * 8;
    if (p.ng > 1 && (split || g.epi == EPI_SWIGLU) && g.sk_cnt && p.kchunks % S == 0 && per_group > 0 &&
        p.tiles * S > per_group && p.tiles * S % per_group != 0 && per_group * p.ng <= kSkCounters) {
        const size_t planes = split ? (size_t)S * g.T * p.vcols : 0;
        const size_t slot_floats = (size_t)256 * sh.MT * 32;
        if (planes + (size_t)per_group * p.ng * slot_floats <= sb.gpart_floats) {
            sk = SK_CONT;
            p.sk_nwg = per_group;
            p.sk_off = planes;
        }
    }
    // slot groups: whole runs of 8 work tiles (one per XCD) for every group
    const int grid = sk == SK_CONT ? p.sk_nwg * p.ng : p.ng == 1 ? p.tiles * S : (p.tiles * S + 7) / 8 * 8 * p.ng;
    if (g.raw) {
        // S partial planes [S][T][N] for a fused consumer to reduce
        hipLaunchKernelGGL(pick(sh, true, EPI_STORE, sk), dim3(grid), dim3(64 * sh.NW), 0, s, p);
    } else if (S == 1) {
        hipLaunchKernelGGL(pick(sh, false, g.epi, sk), dim3(grid), dim3(64 * sh.NW), 0, s, p);
    } else {
        // a split SwiGLU product on four-wave tiles: its last split adds the
        // others' sums (a slot of fp32 accumulators per split and tile) and runs
        // the epilogue, no reduction kernel
        const size_t la_floats = (size_t)p.tiles * S * 128 * sh.MT * 16;  // 128 rows, MT tiles of 16 slots
        const GemmFn la = g.epi == EPI_SWIGLU && g.sk_cnt && p.tiles <= kSkCounters && la_floats <= sb.gpart_floats
                              ? pick_la(sh)
                              : nullptr;
        if (la) {
            hipLaunchKernelGGL(la, dim3(p.tiles * S), dim3(64 * sh.NW), 0, s, p);
            return S;
        }
        hipLaunchKernelGGL(pick(sh, true, g.epi, sk), dim3(grid), dim3(64 * sh.NW), 0, s, p);
        const int ncols = g.epi == EPI_SWIGLU ? p.vcols / 2 : p.vcols;
        const int n = g.T * (ncols / 4);
        hipLaunchKernelGGL(pick_reduce(g.epi), dim3((n + 255) / 256), dim3(256), 0, s, p);
    }
    return S;
}

}  // namespace sdv
