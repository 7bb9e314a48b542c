// Ragged paged causal attention with grouped query heads.
//
// For user b and KV head g the query rows are the (l_b + 1) slots times the
// G query heads sharing g; slot j sits at position i_b + j and attends to
// positions 0 .. i_b + j (cached prefix plus the batch's own earlier slots,
// whose keys the QK-norm/RoPE kernel has already appended to the pages).
//
// bf16 path (MFMA).  A workgroup takes one work item (b, g, context chunk);
// the host sizes chunks so that a batch has about 512 items of equal length.
// The chunk is streamed in 32-token blocks (two KV pages, 16 KB of K and V)
// with direct global-to-LDS loads (one buffer resource over the layer's
// pages, 32-bit offsets) into a ring of LDS buffers, so the next block is in
// flight while one is multiplied, without staging registers.  The block's
// fragments are read from LDS by ds_read instructions issued in inline
// assembly: for reads the compiler sees, it cannot tell a ring buffer from
// the one being loaded and waits for every direct-to-LDS load in flight,
// which leaves nothing in flight during the products (C4 attention 6.1 ->
// 5.5 ms per step); their completion is waited for explicitly.  Each lane
// gathers the piece that belongs to its LDS slot, which leaves the block in
// MFMA fragment order: every operand read is one contiguous 1 KB wave read.
// Wave w owns query-row tiles w, w+4, ... (16 rows each) and, per block:
//   S^T = K Q^T   K rows as the A operand (16 tokens x 32 dims), in the token
//                 order (0-3, 8-11, 16-19, 24-27 | 4-7, 12-15, 20-23, 28-31)
//                 so that each lane ends up with 8 consecutive tokens of one
//                 query row -- the B-operand layout of the next product;
//   O^T += V^T P^T with V^T fragments from the dim-major V page blocks and
//                 P^T taken from registers (no transpose).
// The softmax is online in fp32 (exp2 domain).  Each item writes one partial
// (row max, row sum, unnormalised output); a combine kernel merges the
// partials of a row's chunks in chunk order, so results are deterministic.
//
// fp32 path: one workgroup per (slot, query head), lanes over tokens.
#include "sdv_device.h"
#include "sdv_internal.h"

namespace sdv {

struct AttnP {
    BatchView bv;
    const bf16_t* q;   // [2][T][hq][hd]: hi and lo planes
    KVPool kv;
    int layer;
    int hq, hkv, G;
    float scale_log2;  // log2(e) / sqrt(hd)
    float* apart;      // [items][rows_max][hd]
    float* aml;        // [items][rows_max][2]
    bf16_t* out;       // [2][T][hq][hd]: items that are a user's whole context
};

constexpr int HD = 128;
constexpr int RT_MAX = 2;  // row tiles per wave and pass

// Gather map of the direct-to-LDS block loads.  A block is 32 tokens (two
// pages) of K and V for one KV head, 16 KB, held in LDS as 1024 16-byte
// slots in MFMA fragment order: K slots 0..511, V^T slots 512..1023.  Slot
// s is filled by thread s % 256 of load instruction s / 256, and since a
// wave's direct load writes its 64 lanes to 64 consecutive slots, each lane
// gathers the global piece that belongs to its slot:
//   K slot s: fragment q = s/64 (token half tt = q/4, dim step ds = q%4),
//     lane r = s%64 (lr = r%16, lg = r/16) holds token
//     t = 8*(lr/4) + 4*tt + lr%4 of the block, dims 32*ds + 8*lg .. +7;
//     this token order makes each lane of S^T = K Q^T end up with 8
//     consecutive tokens of one query row (the B layout of O^T += V^T P^T);
//   V slot s: dim tile dt = s/64, r = s%64: dim 16*dt + r%16, tokens
//     8*(r/16 % 2) .. +7 of page r/32 (V pages are dim-major, so this is
//     16 contiguous bytes).
// Returns the page (0/1) of the block and the byte offset inside that
// page's K or V block.
__device__ __forceinline__ void k_slot_src(int s, int& pg, int& off) {
    const int q = s >> 6, r = s & 63;
    const int tt = q >> 2, ds = q & 3, lr = r & 15, lg = r >> 4;
    const int t = 8 * (lr >> 2) + 4 * tt + (lr & 3);
    pg = t >> 4;
    off = ((t & 15) * HD + 32 * ds + 8 * lg) * 2;
}
__device__ __forceinline__ void v_slot_src(int s, int& pg, int& off) {
    const int dt = s >> 6, r = s & 63;
    const int d = 16 * dt + (r & 15), x = r >> 4;
    pg = x >> 1;
    off = (d * kPageTokens + 8 * (x & 1)) * 2;
}

typedef __attribute__((address_space(4))) const int32_t cint32_t;

// Reductions over the four lanes l, l^16, l^32, l^48 that hold one query
// row: each cross-lane swap returns the row halves exchanged between its two
// operands, so combining both results with the own value pairs every lane
// with its partner 16 (then 32) lanes away.
__device__ __forceinline__ float row_max4(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float row_sum4(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Eight 16-byte LDS reads of consecutive 1 KB fragments starting at LDS
// byte address `a` (this lane's slot), issued without a wait.
__device__ __forceinline__ void lds_read8(bf16x8 (&f)[8], uint32_t a) {
    asm volatile(
        "ds_read_b128 %0, %8\n\t"
        "ds_read_b128 %1, %8 offset:1024\n\t"
        "ds_read_b128 %2, %8 offset:2048\n\t"
        "ds_read_b128 %3, %8 offset:3072\n\t"
        "ds_read_b128 %4, %8 offset:4096\n\t"
        "ds_read_b128 %5, %8 offset:5120\n\t"
        "ds_read_b128 %6, %8 offset:6144\n\t"
        "ds_read_b128 %7, %8 offset:7168"
        : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]),
          "=&v"(f[7])
        : "v"(a)
        : "memory");
}

// One 32-token block (its K and V^T fragments) for one row tile.  Scores stay
// in the raw (unscaled) domain until the exponent, which folds the scale in:
// p = 2^(s*c - m*c) with c = log2(e)/sqrt(hd).  Blocks that every row sees
// completely skip the causal/chunk mask; the running output is rescaled only
// when some row's maximum grew; the row sum stays per lane until the end of
// the chunk.  wait_v: called before the first use of the V^T fragments.
template <class F>
__device__ __forceinline__ void attn_block(const bf16x8 (&kfr)[8], const bf16x8 (&vfr)[8], const bf16x8 (&qf)[4],
                                           const bf16x8 (&ql)[4], float& m, float& l, f32x4 (&o)[8], int lim,
                                           int t0, int c1, int lg, bool full, float scale_log2, F wait_v) {
    // S^T = K (Q_hi + Q_lo)^T
    f32x4 sa = f32x4{0.f, 0.f, 0.f, 0.f}, sb = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) {
        const bf16x8 ka = kfr[ds];
        const bf16x8 kk = kfr[4 + ds];
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, qf[ds], sa, 0, 0, 0);
        sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka, ql[ds], sa, 0, 0, 0);
        sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk, qf[ds], sb, 0, 0, 0);
        sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk, ql[ds], sb, 0, 0, 0);
    }
    // lane holds the scores of its query row at tokens t0 + 8*lg + e
    float sc[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        sc[e] = sa[e];
        sc[4 + e] = sb[e];
    }
    if (!full) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int tok = t0 + 8 * lg + e;
            sc[e] = (tok < c1 && tok <= lim) ? sc[e] : -INFINITY;
        }
    }
    float bm = fmaxf(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])),
                     fmaxf(fmaxf(sc[4], sc[5]), fmaxf(sc[6], sc[7])));
    bm = row_max4(bm);
    const float mn = fmaxf(m, bm);
    const bool live = mn != -INFINITY;  // something visible for this row
    const float ms = live ? mn * scale_log2 : 0.f;
    const float alpha = live ? __builtin_amdgcn_exp2f((m - mn) * scale_log2) : 1.f;
    // P as hi + lo bf16 pair (about 16 significant bits)
    float rs = 0.f;
    bf16x8 pb, pl;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float pe = __builtin_amdgcn_exp2f(fmaf(sc[e], scale_log2, -ms));
        rs += pe;
        pb[e] = (__bf16)pe;
        pl[e] = (__bf16)(pe - (float)pb[e]);
    }
    l = fmaf(l, alpha, rs);
    m = mn;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.f)) {
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) o[dt] *= alpha;
    }
    wait_v();
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
        const bf16x8 vf = vfr[dt];
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pb, o[dt], 0, 0, 0);
        o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pl, o[dt], 0, 0, 0);
    }
}

// Per-item constants of the ring and the per-pass state of a wave's row tiles.
struct AttnItem {
    int c0, c1, nblk, prefix, wave, lane, lg, g;
    const cint32_t* pt;
    int kpg0, koff0, kpg1, koff1, vpg0, voff0, vpg1, voff1;  // this thread's gather sources
};
struct AttnState {
    bf16x8 qf[RT_MAX][4], ql[RT_MAX][4];  // query hi / lo planes
    int lim[RT_MAX];
    float m[RT_MAX], l[RT_MAX];
    f32x4 o[RT_MAX][8];
    bool act[RT_MAX];
};

// The chunk's blocks through the LDS ring (buffers r0..r3) for one pass of
// row tiles.
template <int NBUF>
__device__ __forceinline__ void attn_ring(const AttnP& p, const AttnItem& ac, AttnState& st, uint4* r0,
                                          uint4* r1, uint4* r2, uint4* r3) {
    constexpr int PD = NBUF - 1;  // blocks in flight
    static_assert(NBUF >= 2 && NBUF <= 4, "the ring's tail waits cover up to three blocks in flight");
    const int c0 = ac.c0, c1 = ac.c1, nblk = ac.nblk, prefix = ac.prefix, wave = ac.wave;
    const int lane = ac.lane, lg = ac.lg, g = ac.g;
    const int kpg0 = ac.kpg0, koff0 = ac.koff0, kpg1 = ac.kpg1, koff1 = ac.koff1;
    const int vpg0 = ac.vpg0, voff0 = ac.voff0, vpg1 = ac.vpg1, voff1 = ac.voff1;
    const cint32_t* pt = ac.pt;
    auto& qf = st.qf;
    auto& ql = st.ql;
    auto& lim = st.lim;
    auto& m = st.m;
    auto& l = st.l;
    auto& o = st.o;
    auto& act = st.act;
    // One buffer resource over this layer's pages (the host keeps a layer's
    // pages below 4 GB); per lane a 32-bit offset: page * page bytes + the
    // KV head's block + the piece.
    const uint32_t page_bytes = (uint32_t)(p.kv.page_elems() * 2);
    const uint32_t gk = (uint32_t)(p.kv.k_off(0, 0, g) * 2);  // K block of head g
    const uint32_t gv = (uint32_t)(p.kv.v_off(0, 0, g) * 2);  // V block of head g
    const __amdgpu_buffer_rsrc_t kres = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const char*)p.kv.base + p.kv.k_off(p.layer, 0, 0) * 2), (short)0,
        (int)(uint32_t)((uint64_t)p.kv.n_pages * page_bytes), 0x00020000);
    typedef __attribute__((address_space(3))) void lds_void;
    // Requests block blk into LDS buffer buf: four 16-byte direct loads per
    // thread.  Tokens past the chunk end are read from the chunk's last page
    // (the page index is clamped); their scores are masked, and V there is
    // finite (pool zeroed at init, later only model values), so p = 0
    // contributes exactly 0.
    auto issue = [&](int blk, uint4* buf) __attribute__((always_inline)) {
        const int t0 = c0 + blk * 32;
        const uint32_t pb0 = (uint32_t)pt[min(t0, c1 - 1) >> 4] * page_bytes;
        const uint32_t pb1 = (uint32_t)pt[min(t0 + 16, c1 - 1) >> 4] * page_bytes;
        uint4* dst = buf + wave * 64;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kres, (lds_void*)dst, 16, (int)((kpg0 ? pb1 : pb0) + gk + koff0), 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kres, (lds_void*)(dst + 256), 16, (int)((kpg1 ? pb1 : pb0) + gk + koff1), 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kres, (lds_void*)(dst + 512), 16, (int)((vpg0 ? pb1 : pb0) + gv + voff0), 0, 0, 0);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(kres, (lds_void*)(dst + 768), 16, (int)((vpg1 ? pb1 : pb0) + gv + voff1), 0, 0, 0);
    };

    // One 32-token block for this wave's row tiles.
    auto compute = [&](const uint4* buf, int blk) __attribute__((always_inline)) {
        const int t0 = c0 + blk * 32;
        const bool full = t0 + 32 <= c1 && t0 + 31 <= prefix;
        // The block's 16 fragments (8 K, 8 V^T; shared by the wave's row
        // tiles) are read by ds_read instructions the compiler does not see:
        // it cannot tell these reads apart from the direct-to-LDS loads into
        // the other ring buffers and would make them wait for every load in
        // flight.  The reads' completion is waited for explicitly below (the
        // waits take the fragments as operands, so nothing that uses a
        // fragment can be scheduled before its wait).
        bf16x8 kfr[8], vfr[8];
        const uint32_t la = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint4*)buf + lane * 16u;
        lds_read8(kfr, la);
        lds_read8(vfr, la + 512u * 16u);
        asm volatile("s_waitcnt lgkmcnt(8)"
                     : "+v"(kfr[0]), "+v"(kfr[1]), "+v"(kfr[2]), "+v"(kfr[3]), "+v"(kfr[4]),
                       "+v"(kfr[5]), "+v"(kfr[6]), "+v"(kfr[7]));
#pragma unroll
        for (int i = 0; i < RT_MAX; ++i) {
            if (!act[i]) continue;
            attn_block(kfr, vfr, qf[i], ql[i], m[i], l[i], o[i], lim[i], t0, c1, lg, full, p.scale_log2, [&]() {
                if (i == 0)
                    asm volatile("s_waitcnt lgkmcnt(0)"
                                 : "+v"(vfr[0]), "+v"(vfr[1]), "+v"(vfr[2]), "+v"(vfr[3]), "+v"(vfr[4]),
                                   "+v"(vfr[5]), "+v"(vfr[6]), "+v"(vfr[7]));
            });
        }
    };

    // Ring pipeline over NBUF LDS buffers.  Iteration k waits for its own
    // loads of block k (the loads of the blocks issued after it may stay
    // in flight: 4*(PD-1), or 4*(last-k) in the tail) and its LDS reads,
    // then a barrier makes every wave's loads of block k visible and
    // retires every wave's reads of block k-1, whose buffer then
    // receives block k+PD while there is one.  Loads retire in issue
    // order, so the counts are exact; the prologue clamps its block
    // indices (a chunk shorter than PD blocks re-reads its last one,
    // which only makes the waits stricter).
    const int last = nblk - 1;
#pragma unroll
    for (int u = 0; u < PD; ++u) issue(min(u, last), u == 0 ? r0 : u == 1 ? r1 : r2);
    for (int k0 = 0; k0 < nblk; k0 += NBUF) {
#pragma unroll
        for (int u = 0; u < NBUF; ++u) {
            const int k = k0 + u;
            if (k >= nblk) break;
            if (k + PD <= last) {
                wait_vm<4 * (PD - 1), true>();
                barrier_nofence();
                const int nb = (u + PD) % NBUF;
                issue(k + PD, nb == 0 ? r0 : nb == 1 ? r1 : nb == 2 ? r2 : r3);
            } else {
                // tail: blocks k..last are the only ones in flight
                if (last - k >= 2) wait_vm<8, true>();
                else if (last - k == 1) wait_vm<4, true>();
                else wait_vm<0, true>();
                barrier_nofence();
            }
            compute(u == 0 ? r0 : u == 1 ? r1 : u == 2 ? r2 : r3, k);
        }
    }
    // drain the tail loads before the buffers are reused or released
    wait_vm<0>();

}

// Short items of at most two row tiles (attn_item_few: drafting steps, small
// models, short drafts).  They are bound by memory latency, not by bytes: in
// the ring a block is requested when its predecessor's predecessor is done, and
// only as many waves as there are row tiles multiply.  Here the waves share out
// the blocks (one tile: four stripes; two tiles: two stripes, two waves each),
// at most two each, requested at once straight into registers, and merge the
// stripes through LDS.  An item that is a user's whole context writes the
// attention output itself.  bv.few: the host's choice for the batch (every
// context at most five blocks, or at most one item per CU and contexts past 512
// tokens); elsewhere the ring is as fast or faster (a Qwen3-1.7B step of 14
// users of 1000 tokens, 224 an item: 2008 us here, 1972 in the ring).  One user
// of 2000 tokens 1635 -> 1456 us a step, of 1500 1557 -> 1449; 8 users of 134
// tokens, 48 slots, 2052 -> 2005.
__device__ __forceinline__ void attn_few(const AttnP& p, const AttnItem& ac, int item, int b, int R, int tbase,
                                         int ntiles, uint4* r0, uint4* r1, float2 (*ml)[16]) {
    const int wave = ac.wave, lane = ac.lane, lg = ac.lg, lr = lane & 15, g = ac.g;
    const int c0 = ac.c0, c1 = ac.c1, nblk = ac.nblk, prefix = ac.prefix, G = p.G;
    const cint32_t* pt = ac.pt;
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const int ns = ntiles == 1 ? 4 : 2;  // stripes
    const int tile = ntiles == 1 ? 0 : wv & 1, stripe = ntiles == 1 ? wv : wv >> 1;
    const uint32_t page_bytes = (uint32_t)(p.kv.page_elems() * 2);
    const uint32_t gk = (uint32_t)(p.kv.k_off(0, 0, g) * 2), gv = (uint32_t)(p.kv.v_off(0, 0, g) * 2);
    const __amdgpu_buffer_rsrc_t kres = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const char*)p.kv.base + p.kv.k_off(p.layer, 0, 0) * 2), (short)0,
        (int)(uint32_t)((uint64_t)p.kv.n_pages * page_bytes), 0x00020000);
    // lane sources, as k_slot_src / v_slot_src give them: K rows of the two
    // token halves, V^T
    const int kt0 = 8 * (lr >> 2) + (lr & 3), kt1 = kt0 + 4;
    const uint32_t ko0 = gk + (uint32_t)(((kt0 & 15) * HD + 8 * lg) * 2);
    const uint32_t ko1 = gk + (uint32_t)(((kt1 & 15) * HD + 8 * lg) * 2);
    const uint32_t vo = gv + (uint32_t)((lr * kPageTokens + 8 * (lg & 1)) * 2);
    auto load = [&](bf16x8 (&kf)[8], bf16x8 (&vf)[8], int blk) __attribute__((always_inline)) {
        // tokens past the chunk end: the chunk's last page (masked, V finite)
        const int t0 = c0 + blk * 32;
        const uint32_t pb0 = (uint32_t)pt[min(t0, c1 - 1) >> 4] * page_bytes;
        const uint32_t pb1 = (uint32_t)pt[min(t0 + 16, c1 - 1) >> 4] * page_bytes;
        const uint32_t a0 = ko0 + (kt0 >> 4 ? pb1 : pb0), a1 = ko1 + (kt1 >> 4 ? pb1 : pb0);
        const uint32_t av = vo + (lg >> 1 ? pb1 : pb0);
#pragma unroll
        for (int ds = 0; ds < 4; ++ds) {
            kf[ds] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(kres, (int)a0 + 64 * ds, 0, 0));
            kf[4 + ds] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(kres, (int)a1 + 64 * ds, 0, 0));
        }
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
            vf[dt] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(kres, (int)av + 512 * dt, 0, 0));
    };
    const int row = tile * 16 + lr;
    const bool ok = row < R;
    const int j = ok ? row / G : 0, hh = ok ? row % G : 0;
    const bf16_t* qs = p.q + ((size_t)(tbase + j) * p.hq + g * G + hh) * HD + 8 * lg;
    const size_t qpl = (size_t)p.bv.T * p.hq * HD;
    bf16x8 qf[4], ql[4], ka[8], va[8], kb[8], vb[8];
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) {
        qf[ds] = *(const bf16x8*)(qs + ds * 32);  // rows past R: the first row's (their outputs are not stored)
        ql[ds] = *(const bf16x8*)(qs + qpl + ds * 32);
    }
    if (stripe < nblk) load(ka, va, stripe);
    if (stripe + ns < nblk) load(kb, vb, stripe + ns);
    __builtin_amdgcn_sched_barrier(0);
    const int lim = prefix + j;
    float m = -INFINITY, l = 0.f;
    f32x4 o[8];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto block = [&](const bf16x8 (&kf)[8], const bf16x8 (&vf)[8], int k) __attribute__((always_inline)) {
        const int t0 = c0 + k * 32;
        attn_block(kf, vf, qf, ql, m, l, o, lim, t0, c1, lg, t0 + 32 <= c1 && t0 + 31 <= prefix, p.scale_log2, [] {});
    };
    if (stripe < nblk) block(ka, va, stripe);
    if (stripe + ns < nblk) block(kb, vb, stripe + ns);
    const float lsum = row_sum4(l);
    f32x4* os = (f32x4*)((wave < 2 ? r0 : r1) + (wave & 1) * 512);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) os[dt * 64 + lane] = o[dt];
    if (lg == 0) ml[wave][lr] = float2{m == -INFINITY ? -INFINITY : m * p.scale_log2, lsum};
    __syncthreads();
    const int i0 = p.bv.item_off[b];
    const bool solo = p.bv.item_off[b + 1] - i0 == p.hkv;
    // piece (tile, dt, lane) of 16 bytes: row lane % 16, dims 16 * dt + 4 * (lane / 16) ..
    for (int e = threadIdx.x; e < ntiles * 512; e += 256) {
        const int tl = e >> 9, dt = (e >> 6) & 7, ln = e & 63, rr = ln & 15, orow = tl * 16 + rr;
        if (orow >= R) continue;
        float M = -INFINITY;
        for (int s = 0; s < ns; ++s) M = fmaxf(M, ml[ntiles == 1 ? s : 2 * s + tl][rr].x);
        f32x4 a = f32x4{0.f, 0.f, 0.f, 0.f};
        float L = 0.f;
        for (int s = 0; s < ns; ++s) {  // stripe order
            const int w = ntiles == 1 ? s : 2 * s + tl;
            const float2 v = ml[w][rr];
            const float f = v.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(v.x - M);
            L += v.y * f;
            a += ((const f32x4*)((w < 2 ? r0 : r1) + (w & 1) * 512))[dt * 64 + ln] * f;
        }
        const int d0 = dt * 16 + 4 * (ln >> 4);
        if (solo) {
            const float inv = 1.0f / L;
            const float ov[4] = {a[0] * inv, a[1] * inv, a[2] * inv, a[3] * inv};
            const int jj = orow / G;
            st_act4(p.out, qpl, ((size_t)(tbase + jj) * p.hq + g * G + orow % G) * HD + d0, ov);
        } else {
            const size_t pr = (size_t)item * p.bv.rows_max + orow;
            *(f32x4*)(p.apart + pr * HD + d0) = a;
            if (d0 == 0) *(float2*)(p.aml + pr * 2) = float2{M, L};
        }
    }
}

template <int NBUF>
__device__ __forceinline__ void attn_bf16_body(const AttnP& p, uint4* r0, uint4* r1, uint4* r2, uint4* r3,
                                               float2 (*ml)[16]) {
    // The batch metadata is read-only while the kernel runs: reading it
    // through the constant address space gives scalar loads, which keep the
    // vector memory counter (waited on below) free of anything but KV.
    const cint32_t* items = (const cint32_t*)p.bv.items;
    const int item = blockIdx.x;
    const int b = items[4 * item + 0], g = items[4 * item + 1];
    const int c0 = items[4 * item + 2], c1 = items[4 * item + 3];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lr = lane & 15, lg = lane >> 4;
    const int G = p.G;
    const int R = (((const cint32_t*)p.bv.L)[b] + 1) * G;
    const int prefix = ((const cint32_t*)p.bv.prefix)[b];
    const int tbase = ((const cint32_t*)p.bv.slot_off)[b];
    const cint32_t* pt = (const cint32_t*)p.bv.page_table + (size_t)b * p.bv.max_pages;
    const int nblk = (c1 - c0 + 31) >> 5;

    // this thread's four gather sources (page of the block, byte offset)
    int kpg0, koff0, kpg1, koff1, vpg0, voff0, vpg1, voff1;
    k_slot_src(threadIdx.x, kpg0, koff0);
    k_slot_src(256 + threadIdx.x, kpg1, koff1);
    v_slot_src(threadIdx.x, vpg0, voff0);
    v_slot_src(256 + threadIdx.x, vpg1, voff1);
    AttnItem ac;
    ac.c0 = c0;
    ac.c1 = c1;
    ac.nblk = nblk;
    ac.prefix = prefix;
    ac.wave = wave;
    ac.lane = lane;
    ac.lg = lg;
    ac.g = g;
    ac.pt = pt;
    ac.kpg0 = kpg0; ac.koff0 = koff0; ac.kpg1 = kpg1; ac.koff1 = koff1;
    ac.vpg0 = vpg0; ac.voff0 = voff0; ac.vpg1 = vpg1; ac.voff1 = voff1;
    const int ntiles = (R + 15) >> 4;
    if (p.bv.few && attn_item_few(R, nblk)) {
        attn_few(p, ac, item, b, R, tbase, ntiles, r0, r1, ml);
        return;
    }
    for (int rp = 0; rp < ntiles; rp += 4 * RT_MAX) {
        // this wave's row tiles in this pass: rp + wave + 4*i
        AttnState st;
        auto& qf = st.qf;  // query hi / lo planes
        auto& ql = st.ql;
        auto& lim = st.lim;
        auto& m = st.m;
        auto& l = st.l;
        auto& o = st.o;
        auto& act = st.act;
#pragma unroll
        for (int i = 0; i < RT_MAX; ++i) {
            const int tile = rp + wave + 4 * i;
            act[i] = tile < ntiles;
            const int row = tile * 16 + lr;
            const bool ok = act[i] && row < R;
            const int j = ok ? row / G : 0, hh = ok ? row % G : 0;
            const bf16_t* qs = p.q + ((size_t)(tbase + j) * p.hq + g * G + hh) * HD + 8 * lg;
            const size_t qpl = (size_t)p.bv.T * p.hq * HD;
#pragma unroll
            for (int ds = 0; ds < 4; ++ds) {
                qf[i][ds] = ok ? *(const bf16x8*)(qs + ds * 32) : bf16x8{};
                ql[i][ds] = ok ? *(const bf16x8*)(qs + qpl + ds * 32) : bf16x8{};
            }
            lim[i] = prefix + j;
            m[i] = -INFINITY;
            l[i] = 0.f;
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) o[i][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        // the query loads must not be counted by the block waits below
        wait_vm<0>();

        attn_ring<NBUF>(p, ac, st, r0, r1, r2, r3);

        // partial of this item: lane holds O^T[d = dt*16 + 4*lg + r][row lr]
#pragma unroll
        for (int i = 0; i < RT_MAX; ++i) {
            if (!act[i]) continue;
            const int row = (rp + wave + 4 * i) * 16 + lr;
            const float lsum = row_sum4(l[i]);  // all lanes take part in the swaps
            if (row >= R) continue;
            const size_t pr = (size_t)item * p.bv.rows_max + row;
            if (lg == 0) {
                p.aml[pr * 2 + 0] = m[i] == -INFINITY ? -INFINITY : m[i] * p.scale_log2;
                p.aml[pr * 2 + 1] = lsum;
            }
#pragma unroll
            for (int dt = 0; dt < 8; ++dt)
                *(f32x4*)(p.apart + pr * HD + dt * 16 + 4 * lg) = o[i][dt];
        }
        __syncthreads();  // the LDS buffers are reused by the next row pass
    }
}

template <int NBUF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_attn_bf16(AttnP p) {
    __shared__ __attribute__((aligned(16))) uint4 kv0[1024];
    __shared__ __attribute__((aligned(16))) uint4 kv1[1024];
    __shared__ __attribute__((aligned(16))) uint4 kv2[NBUF > 2 ? 1024 : 1];
    __shared__ __attribute__((aligned(16))) uint4 kv3[NBUF > 3 ? 1024 : 1];
    __shared__ float2 ml[4][16];
    attn_bf16_body<NBUF>(p, kv0, kv1, kv2, kv3, ml);
}

// Merge the partials of the chunks of (b, g) for one query row in chunk
// order; half a wave per (slot, query head), lane l of it holding dims
// 4l..4l+3 (16-byte partial loads, 8-byte stores of the two output planes).
// Chunks are taken eight at a time with all their loads issued before the
// merge (online maximum: the running sums are rescaled when a group raises
// it).
__global__ __launch_bounds__(256) void k_attn_combine(BatchView bv, const float* apart,
                                                      const float* aml, bf16_t* out, int hq, int hkv) {
    const int rid = blockIdx.x * 8 + (threadIdx.x >> 5);  // (slot, query head)
    const int l = threadIdx.x & 31;
    const int t = rid / hq, h = rid % hq;
    if (t >= bv.T) return;
    const int G = hq / hkv, g = h / G, hh = h % G;
    const int b = bv.slot_b[t], j = bv.slot_j[t];
    const int row = j * G + hh;
    const int i0 = bv.item_off[b], nch = (bv.item_off[b + 1] - i0) / hkv;
    // a short context in one item: the item wrote the output
    if (nch == 1 && bv.few && attn_item_few((bv.L[b] + 1) * G, (bv.prefix[b] + bv.L[b] + 32) >> 5)) return;
    const int p0 = i0 + g * nch, p1 = p0 + nch;
    float M = -INFINITY, Ls = 0.f;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int pg = p0; pg < p1; pg += 8) {
        float mi[8], li[8];
        f32x4 a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool ok = pg + u < p1;
            const size_t pr = (size_t)(ok ? pg + u : p0) * bv.rows_max + row;
            mi[u] = ok ? aml[pr * 2] : -INFINITY;
            li[u] = ok ? aml[pr * 2 + 1] : 0.f;
            a[u] = ok ? *(const f32x4*)(apart + pr * HD + 4 * l) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
        float mg = M;
#pragma unroll
        for (int u = 0; u < 8; ++u) mg = fmaxf(mg, mi[u]);
        if (mg == -INFINITY) continue;  // no key of these chunks is visible to the row
        const float sc = exp2f(M - mg);  // 0 while M is still -inf
        Ls *= sc;
        acc *= sc;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            if (mi[u] == -INFINITY) continue;
            const float w = exp2f(mi[u] - mg);
            Ls += li[u] * w;
            acc += a[u] * w;
        }
        M = mg;
    }
    const float inv = 1.0f / Ls;
    const float o[4] = {acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
    st_act4(out, (size_t)bv.T * hq * HD, ((size_t)t * hq + h) * HD + 4 * l, o);
}

// fp32 path: one workgroup per (slot, query head); its four waves take every
// fourth block of 64 tokens and are merged in wave order.  Scores: lane =
// token (its key row in 16-byte pieces where rows are aligned); the softmax is
// online per block, one pair of wave reductions per 64 tokens; outputs: lane =
// dim, the 64 weights broadcast from LDS against the dim-major value blocks.
// (One wave per row with a reduction per token took 98 us for 113 tokens of
// four heads and 16 slots; this takes 7.4.)
template <bool VEC>
__global__ __launch_bounds__(256) void k_attn_f32(BatchView bv, const float* q, KVPool kv,
                                                  int layer, float* out, int hq, int hkv, int hd,
                                                  float scale) {
    __shared__ float qs[128];
    __shared__ __attribute__((aligned(16))) float ps[4][64];
    __shared__ float ms[4], ls[4], os[4][128];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int t = blockIdx.x / hq, h = blockIdx.x % hq;
    const int G = hq / hkv, g = h / G;
    const int b = bv.slot_b[t];
    const int n = bv.prefix[b] + bv.slot_j[t] + 1;
    const int32_t* pt = bv.page_table + (size_t)b * bv.max_pages;
    const float* base = (const float*)kv.base;
    if (threadIdx.x < hd) qs[threadIdx.x] = q[((size_t)t * hq + h) * hd + threadIdx.x];
    __syncthreads();
    float m = -INFINITY, l = 0.f, a0 = 0.f, a1 = 0.f;
    for (int c0 = wave * 64; c0 < n; c0 += 256) {
        const int tok = c0 + lane;
        float d = -INFINITY;
        if (tok < n) {
            const float* kr = base + kv.k_off(layer, pt[tok >> 4], g) + (size_t)(tok & 15) * hd;
            float s = 0.f;
            if (VEC) {
                for (int a = 0; a < hd; a += 4) {
                    const f32x4 v = *(const f32x4*)(kr + a);
#pragma unroll
                    for (int e = 0; e < 4; ++e) s = fmaf(qs[a + e], v[e], s);
                }
            } else {
                for (int a = 0; a < hd; ++a) s = fmaf(qs[a], kr[a], s);
            }
            d = s * scale;
        }
        const float mn = fmaxf(m, wave_max(d));
        const float al = expf(m - mn), pe = expf(d - mn);
        l = l * al + wave_sum(pe);
        m = mn;
        a0 *= al;
        a1 *= al;
        wave_lds_order();     // the previous block's weights have been read
        ps[wave][lane] = pe;  // read back by the same wave
        wave_lds_order();
        const int nt = min(64, n - c0);
        for (int p0 = 0; p0 < nt; p0 += kPageTokens) {
            const float* vb = base + kv.v_off(layer, pt[(c0 + p0) >> 4], g);
#pragma unroll
            for (int u = 0; u < kPageTokens; u += 4) {
                const f32x4 pv = *(const f32x4*)&ps[wave][p0 + u];
                const f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
                const f32x4 v0 = lane < hd ? *(const f32x4*)(vb + (size_t)lane * kPageTokens + u) : z;
                const f32x4 v1 = lane + 64 < hd ? *(const f32x4*)(vb + (size_t)(lane + 64) * kPageTokens + u) : z;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (p0 + u + e >= nt) continue;  // rows past the context may hold anything
                    a0 = fmaf(pv[e], v0[e], a0);
                    a1 = fmaf(pv[e], v1[e], a1);
                }
            }
        }
    }
    if (lane == 0) {
        ms[wave] = m;
        ls[wave] = l;
    }
    os[wave][lane] = a0;
    os[wave][lane + 64] = a1;
    __syncthreads();
    if ((int)threadIdx.x >= hd) return;
    const float M = fmaxf(fmaxf(ms[0], ms[1]), fmaxf(ms[2], ms[3]));
    float L = 0.f, o = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const float f = expf(ms[w] - M);  // 0 for a wave without tokens
        L += ls[w] * f;
        o += os[w][threadIdx.x] * f;
    }
    out[((size_t)t * hq + h) * hd + threadIdx.x] = o / L;
}

void launch_attention(const Dims& D, const BatchView& bv, const SlotBufs& sb, const KVPool& kv,
                      int layer, hipStream_t s) {
    if (!D.bf16) {
        // key rows of a multiple of 4 floats start on 16 bytes (the pool is
        // 256-byte aligned)
        const auto fn = D.hd % 4 == 0 ? k_attn_f32<true> : k_attn_f32<false>;
        hipLaunchKernelGGL(fn, dim3(bv.T * D.hq), dim3(256), 0, s, bv, (const float*)sb.qbuf, kv, layer,
                           (float*)sb.attn, D.hq, D.hkv, D.hd, 1.0f / sqrtf((float)D.hd));
        return;
    }
    AttnP p;
    p.bv = bv;
    p.q = (const bf16_t*)sb.qbuf;
    p.kv = kv;
    p.layer = layer;
    p.hq = D.hq;
    p.hkv = D.hkv;
    p.G = D.G();
    p.scale_log2 = 1.4426950408889634f / sqrtf((float)D.hd);
    p.apart = sb.apart;
    p.aml = sb.aml;
    p.out = (bf16_t*)sb.attn;
    hipLaunchKernelGGL(k_attn_bf16<kAttnBuffers>, dim3(bv.n_items), dim3(256), 0, s, p);
    // half a wave per (slot, query head)
    if (!bv.combine) return;
    hipLaunchKernelGGL(k_attn_combine, dim3((bv.T * D.hq + 7) / 8), dim3(256), 0, s, bv, sb.apart,
                       sb.aml, (bf16_t*)sb.attn, D.hq, D.hkv);
}

}  // namespace sdv
