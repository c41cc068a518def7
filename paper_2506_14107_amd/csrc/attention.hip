// Attention over mixed fresh and reference K/V.
//
// Each key row is read through pos[]: a recomputed token's own packed row, or -- for a reused token
// -- the packed row of the same token of the frame it is reused from.  Three bf16 kernels share one
// softmax loop (attend_tile), one query tile of 32 per wavefront:
//   streamed (attn_stream_k)   four tiles of a frame and head per block, keys through a small LDS ring
//   per frame (attn_mfma_k)    all keys of a frame and head in LDS, its tiles over eight wavefronts
//   per unit (attn_unit_k)     star groups: the reference's keys in LDS once for a group's frames
// attn_plan.h says which runs when, and why.
//
// bf16 path (MFMA 32x32x16, fp32 accumulate), every quantity kept with one query per lane:
//   S^T = K . Q^T      A = K rows from LDS, B = the query tile (registers); lane l holds the
//                      scores of query l%32 against 16 of the 32 keys of a key block
//   online softmax     max / sum over a lane's 16 registers plus one shuffle with lane l^32
//   O^T += V^T . P^T   A = V^T, read from row-major V with the transposing LDS read
//                      ds_read_b64_tr_b16; B = the probabilities as they sit in the S^T
//                      accumulators; the contraction runs over the 32 keys in the order the
//                      accumulator layout gives (the same order on both operands)
// so a lane rescales and normalises its own query's output without any shuffle.  A query tile is
// always taken by one wavefront over all key blocks in order, whatever kernel runs it and however
// many other queries its frame has, so a row's result depends only on its query and the frame's
// keys and values (no split of the keys across wavefronts, whose merge would round the
// probabilities against partial maxima).
//
// fp32 path: the same products on v_mfma_f32_16x16x4_f32 (attn_f32_k).
#include <algorithm>
#include <type_traits>

#include "attn_plan.h"

namespace dv {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Workgroup barrier that orders LDS only: this wave's LDS operations are complete and every
// wave has arrived.  Unlike __syncthreads() it does not wait for global stores in flight, so
// the output rows of one work item drain while the next item is staged.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

__device__ inline float wmax(float v) {
    for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ inline float wsum(float v) {
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// four floats to four bf16 (round to nearest even, v_cvt_pk_bf16_f32)
__device__ inline uint2 pack_bf16x4(float a, float b, float c, float d) {
    const bf16x4 v = {(__bf16)a, (__bf16)b, (__bf16)c, (__bf16)d};
    return __builtin_bit_cast(uint2, v);
}
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));   // native vector: stays in VGPRs

// The value a lane's partner in the other half of the wavefront (lane l ^ 32) holds.
__device__ inline float other_half(float x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __builtin_bit_cast(float, (threadIdx.x & 32) ? r[0] : r[1]);
}

constexpr int AW = 8;    // wavefronts of a per-frame attention block
constexpr int UW = 12;   // wavefronts of a per-unit attention block

// Online-softmax attention of one query tile (fragments qf, one query per lane) against the
// staged K/V: key blocks taken two at a time in order (kb, kb + 1) -- two independent MFMA
// chains and at most one rescale per step.  krow maps a key to its LDS row; stage(kb) runs
// before the step of blocks kb, kb + 1 reads them (a kernel streaming K/V through LDS loads them
// there).  On return (m, l, o) hold the maximum the tile's probabilities are scaled to (raw score
// units; at most 8 / sl2 below the running maximum), their sum and the unnormalised output.  The
// arithmetic and its order depend only on the key values, never on where the rows sit.
template <int DH, class KRow, class Stage>
__device__ __forceinline__ void attend_tile(const Geo& g, const uint16_t* Ks, const uint16_t* Vs,
                                            int N, int lane, const bf16x8 (&qf)[DH / 16],
                                            KRow krow, float& m, float& l,
                                            f32x16 (&o)[(DH + 31) / 32], Stage stage) {
    constexpr int KS = DH / 16;          // k-steps of S^T
    constexpr int DB = (DH + 31) / 32;   // 32-row blocks of O^T
    const int hl = lane >> 5, lr = lane & 31;
    const float sl2 = 1.4426950408889634f / sqrtf((float)DH);  // log2(e) / sqrt(dh)
    const float lazy = 8.0f / sl2;    // raw score units of a factor 2^8
    const int nkb = g.npad / 32;
    const int grp = lane >> 4, gi = lane & 15;    // 16-lane group of the transposing read
    const int tr_key = hl * 4 + (gi >> 2);
    const int tr_dim = (grp & 1) * 16 + (gi & 3) * 4;

    // scores of key block kb against the query tile (raw, unscaled); MK: the block may hold
    // keys past N
    auto scores = [&](int kb, auto mk) {
        f32x16 sc;
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = 0.f;
        const int row = krow(kb * 32 + lr);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 kf = *(const bf16x8*)(Ks + g.kofs(row, ks * 2 + hl));
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], sc, 0, 0, 0);
        }
        if (decltype(mk)::value && (kb + 1) * 32 > N) {   // ragged last block: keys past N get -inf
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = kb * 32 + (r >> 2) * 8 + hl * 4 + (r & 3);
                sc[r] = key < N ? sc[r] : -INFINITY;
            }
        }
        return sc;
    };
    // O^T += V^T(kb) . P^T(kb)
    auto accumulate = [&](int kb, const bf16x8 (&pf)[2]) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            // lane (group grp, index gi) names key kb*32 + ks*16 + hl*4 + gi/4 (+8) and dims
            // b*32 + (grp&1)*16 + 4*(gi%4); it receives dim b*32 + (grp&1)*16 + gi of the 4
            // keys named by lanes 4e + gi/4 of its group
            const int key = kb * 32 + ks * 16 + tr_key;
            const int r0 = krow(key), r1 = krow(key + 8);
#pragma unroll
            for (int b = 0; b < DB; ++b) {
                int d = b * 32 + tr_dim;
                d = d < DH ? d : DH - 4;   // head dims past DH: any finite row data
                const uint16_t* p0 = Vs + g.vofs(r0, d >> 3) + (d & 7);
                const uint16_t* p1 = Vs + g.vofs(r1, d >> 3) + (d & 7);
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4*)p0);
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4*)p1);
                const s16x4 both[2] = {lo, hi};
                const bf16x8 vf = __builtin_bit_cast(bf16x8, both);
                o[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[ks], o[b], 0, 0, 0);
            }
        }
    };

#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
    m = -INFINITY;
    l = 0.f;
    // One softmax step over key blocks kb and kb + 1.  MK: the step may hold the ragged last
    // block or no second block; only the loop's tail steps do, so the others carry no per-key
    // test (the arithmetic and its order are the same either way).
    auto step = [&](int kb, auto mk) {
        constexpr bool MK = decltype(mk)::value;
        stage(kb);
        const int kb1 = kb + 1;
        const bool two = !MK || kb1 < nkb;
        const f32x16 s0 = scores(kb, mk);
        f32x16 s1;
        if (two) {
            s1 = scores(kb1, mk);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) s1[r] = -INFINITY;
        }
        // block maximum and, below, the probability sum as pairwise trees (short dependency
        // chains; the maximum is exact in any order)
        float mx[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) mx[r] = fmaxf(s0[r], s1[r]);
#pragma unroll
        for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
            for (int r = 0; r < w; ++r) mx[r] = fmaxf(mx[r], mx[r + w]);
        float bm = mx[0];
        bm = fmaxf(bm, other_half(bm));
        // rescale only when some lane's block maximum passes its reference maximum m by more
        // than 8 in log2 units: probabilities stay below 2^8 (far inside the range of the fp32
        // sums and bf16 products), and most steps after the first keep their scale
        if (__any(bm > m + lazy)) {
            const float mn = fmaxf(m, bm);
            const float alpha = __builtin_amdgcn_exp2f((m - mn) * sl2);
            l *= alpha;
#pragma unroll
            for (int b = 0; b < DB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) o[b][r] *= alpha;
            m = mn;
        }
        const float nm = -m * sl2;
        float sr[16];
        bf16x8 p0[2], p1[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float e0 = __builtin_amdgcn_exp2f(fmaf(s0[r], sl2, nm));
            const float e1 = __builtin_amdgcn_exp2f(fmaf(s1[r], sl2, nm));
            sr[r] = e0 + e1;
            p0[r >> 3][r & 7] = (__bf16)e0;
            p1[r >> 3][r & 7] = (__bf16)e1;
        }
#pragma unroll
        for (int w = 8; w >= 1; w >>= 1)
#pragma unroll
            for (int r = 0; r < w; ++r) sr[r] += sr[r + w];
        const float ps = sr[0];
        l += ps + other_half(ps);
        accumulate(kb, p0);
        if (two) accumulate(kb1, p1);
    };
    const int nfull = N / 32;   // key blocks with no key past N
    int kb = 0;
    for (; kb + 1 < nfull; kb += 2) step(kb, std::integral_constant<bool, false>());
    for (; kb < nkb; kb += 2) step(kb, std::integral_constant<bool, true>());
}

// o / l of a lane's query as bf16 to its output row (dims of this lane's register groups)
template <int DH>
__device__ __forceinline__ void store_row(uint16_t* dst, int lane, float l,
                                          const f32x16 (&o)[(DH + 31) / 32]) {
    constexpr int DB = (DH + 31) / 32;
    const int hl = lane >> 5;
    const float inv = 1.0f / l;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const int d = b * 32 + q4 * 8 + hl * 4;
            if (d < DH)
                *(uint2*)(dst + d) = pack_bf16x4(o[b][q4 * 4 + 0] * inv, o[b][q4 * 4 + 1] * inv,
                                                 o[b][q4 * 4 + 2] * inv, o[b][q4 * 4 + 3] * inv);
        }
}

// ---- per-frame items ---------------------------------------------------------------------------
// Work split: T = ceil(q/32) query tiles over AW wavefronts, each tile over all key blocks.
template <int DH>
__device__ __forceinline__ void attn_item(const AttnArgs& a, int f, int h, char* smem);

template <int DH>
__global__ __launch_bounds__(AW * 64) __attribute__((amdgpu_waves_per_eu(DH == 64 ? 4 : 2, DH == 64 ? 4 : 2)))
void attn_mfma_k(AttnArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    // The grid holds as many blocks as are resident at once and each block walks a list of work
    // items (frame f, head h), heads fastest: one item per launch slot would leave the compute
    // units waiting on workgroup dispatch when items are short.
    for (int item = blockIdx.x; item < a.F * a.H; item += gridDim.x) {
        attn_item<DH>(a, item / a.H, item % a.H, smem);
        lds_barrier();   // the next item restages K/V over this item's LDS
    }
}

// One work item: frame f, head h.  Every thread of the block takes the same path.
template <int DH>
__device__ __forceinline__ void attn_item(const AttnArgs& a, int f, int h, char* smem) {
    constexpr int KS = DH / 16;          // k-steps of S^T
    constexpr int DB = (DH + 31) / 32;   // 32-row blocks of O^T
    constexpr int CH = DH / 8;           // 16-byte chunks per row
    constexpr int NT = AW * 64;
    const int N = a.N, D = a.D;
    const Geo g(N, DH);
    uint16_t* Ks = (uint16_t*)smem;
    uint16_t* Vs = Ks + (size_t)g.npad * g.ldk;
    // the thread index passes through an empty asm so that nothing derived from it is hoisted
    // out of the caller's item loop (that would keep it live, and spilled, across items)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = tid >> 6;
    const int hl = lane >> 5, lr = lane & 31;
    const size_t ld3 = 3 * (size_t)D;
    const uint16_t* qkv = (const uint16_t*)a.qkv;
    const int q0 = a.qoff[f], q1 = a.qoff[f + 1];
    const int ntile = (q1 - q0 + 31) / 32;
    if (ntile == 0) return;

    // stage K and V rows (row-major, 16-byte chunks); keys past N repeat key N-1 (finite data
    // whose scores are masked).  Up to SU chunks per thread are gathered before any store
    // (257 keys of head dim 64 in one pass).
    constexpr int SU = 5;
    const int total = g.npad * CH;
    // the first tile's queries are requested ahead of the keys
    auto load_q = [&](int t, bf16x8 (&qf)[KS]) {
        const int myq = q0 + t * 32 + lr;
        const int qrow = myq < q1 ? myq : q1 - 1;   // tail lanes compute on a valid row
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qf[ks] = *(const bf16x8*)(qkv + (size_t)qrow * ld3 + h * DH + ks * 16 + hl * 8);
    };
    bf16x8 qf[KS];
    load_q(wave, qf);
    for (int c0 = tid; c0 < total; c0 += SU * NT) {
        size_t rowoff[SU];
        u32x4 kv[SU], vv[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int c = min(c0 + u * NT, total - 1);
            const int j = min(c / CH, N - 1);
            rowoff[u] = (size_t)a.pos[(size_t)f * N + j] * ld3 + h * DH + (c % CH) * 8;
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            kv[u] = *(const u32x4*)(qkv + rowoff[u] + D);
            vv[u] = *(const u32x4*)(qkv + rowoff[u] + 2 * D);
        }
#pragma unroll
        for (int u = 0; u < SU; ++u) {
            const int c = c0 + u * NT;
            if (c < total) {
                const int j = c / CH, part = c % CH;
                *(u32x4*)(Ks + g.kofs(j, part)) = kv[u];
                *(u32x4*)(Vs + g.vofs(j, part)) = vv[u];
            }
        }
    }
    lds_barrier();

    float m, l;   // the probabilities' scale (raw score units) and their sum
    f32x16 o[DB];
    for (int t = wave; t < ntile; t += AW) {
        if (t != wave) load_q(t, qf);
        const int myq = q0 + t * 32 + lr;
        attend_tile<DH>(g, Ks, Vs, N, lane, qf, [](int k) { return k; }, m, l, o, [](int) {});
        if (myq < q1) store_row<DH>((uint16_t*)a.out + (size_t)myq * D + h * DH, lane, l, o);
    }
}

// ---- streamed items ----------------------------------------------------------------------------
// A block of four wavefronts takes up to four query tiles of a frame and head and streams the
// frame's keys and values through a two-buffer ring of 64 keys (one step of attend_tile): a step's
// rows wait in registers while the step before is computed, then go to LDS behind one barrier.  The
// ring is small, so several blocks share a compute unit and one's barriers and load latency are
// partly covered by the others' arithmetic.  The softmax's VALU work is the largest part (577 keys, 60 %
// reuse: about 108 us a layer for 128 frames at 1336 VALU cycles a step, of 168 measured); the rest is
// latency that three wavefronts per SIMD leave open.  Two or eight wavefronts a block, or registers for
// a fourth wavefront per SIMD, were slower or equal.
template <int DH>
__global__ __launch_bounds__(FW * 64) __attribute__((amdgpu_waves_per_eu(DH == 64 ? 3 : 2, DH == 64 ? 3 : 2)))
void attn_stream_k(AttnArgs a, StreamMap map) {
    constexpr int KS = DH / 16;
    constexpr int DB = (DH + 31) / 32;
    constexpr int CH = DH / 8;                       // 16-byte chunks per row
    constexpr int NT = FW * 64;
    constexpr int PC = (64 * CH + NT - 1) / NT;      // chunks of K (and of V) per thread and step
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int N = a.N, D = a.D;
    const Geo g(N, DH);
    uint16_t* Ks = (uint16_t*)smem;
    uint16_t* Vs = Ks + (size_t)128 * g.ldk;
    // both cache lines of the arguments are requested before either is used (a serial miss costs 0.2 us)
    const int* qoff = a.qoff;
    int span = map.span;
    asm volatile("" : "+s"(qoff), "+s"(span));
    int f, h, qb;
    if (!map.item(blockIdx.x, f, h, qb)) return;
    const int q0 = qoff[f], q1 = qoff[f + 1];
    const int ntile = (q1 - q0 + 31) / 32;
    const int nb = (ntile + FW - 1) / FW;            // blocks the tiles are dealt to
    if (qb >= nb) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int hl = lane >> 5, lr = lane & 31;
    const size_t ld3 = 3 * (size_t)D;
    const uint16_t* qkv = (const uint16_t*)a.qkv + (size_t)h * DH;
    const int t = qb + wave * nb;
    const int myq = q0 + t * 32 + lr;
    const int qrow = myq < q1 ? myq : q1 - 1;        // tail lanes compute on a valid row
    bf16x8 qf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        qf[ks] = *(const bf16x8*)(qkv + (size_t)qrow * ld3 + ks * 16 + hl * 8);

    const int* pos = a.pos + (size_t)f * N;
    // the packed rows are below 2^32 bytes and 2^24 in number: 32-bit byte offsets, 24-bit products
    const auto rq = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.qkv), (short)0,
                                                      (int)0xFFFFFFF0u, 0x00020000);
    uint32_t prow[PC], kofs[PC], vofs[PC], coff[PC];
    int key[PC];
#pragma unroll
    for (int p = 0; p < PC; ++p) {
        const int i = min(tid + p * NT, 64 * CH - 1), r = i / CH, c = i % CH;
        key[p] = r;
        kofs[p] = g.kofs(r, c);
        vofs[p] = g.vofs(r, c);
        coff[p] = (h * DH + D + c * 8) * 2;
    }
    u32x4 kv[PC], vv[PC];
    auto rows = [&](int k0) {   // packed rows of keys k0 .. k0 + 63 (past N: key N - 1, masked)
#pragma unroll
        for (int p = 0; p < PC; ++p) prow[p] = pos[min(k0 + key[p], N - 1)];
    };
    auto load = [&]() {
#pragma unroll
        for (int p = 0; p < PC; ++p) {
            const uint32_t off = __umul24(prow[p], 6 * D) + coff[p];
            kv[p] = __builtin_amdgcn_raw_buffer_load_b128(rq, (int)off, 0, 0);
            vv[p] = __builtin_amdgcn_raw_buffer_load_b128(rq, (int)off, 2 * D, 0);
        }
    };
    rows(0);
    load();
    rows(64);
    // before the step of keys k0 .. k0 + 63: every wave has finished the step two before (it passed
    // the last barrier after it), so that step's buffer is free
    auto stage = [&](int kb) {
        const int k0 = kb * 32;
        uint16_t* const Kb = Ks + (k0 & 64) * g.ldk;
        uint16_t* const Vb = Vs + (k0 & 64) * g.ldv;
#pragma unroll
        for (int p = 0; p < PC; ++p)
            if (64 * CH % NT == 0 || tid + p * NT < 64 * CH) {
                *(u32x4*)(Kb + kofs[p]) = kv[p];
                *(u32x4*)(Vb + vofs[p]) = vv[p];
            }
        if (k0 + 64 < N) {
            load();
            rows(k0 + 128);
        }
        lds_barrier();
    };
    if (t < ntile) {
        float m, l;
        f32x16 o[DB];
        attend_tile<DH>(g, Ks, Vs, N, lane, qf, [](int k) { return k & 127; }, m, l, o, stage);
        if (myq < q1) store_row<DH>((uint16_t*)a.out + (size_t)myq * D + h * DH, lane, l, o);
    } else {
        for (int kb = 0; kb < g.npad / 32; kb += 2) stage(kb);   // the block's barriers and copies
    }
}

template <int DH>
void launch_stream(const AttnArgs& a, hipStream_t s) {
    const Geo g(a.N, DH);
    const size_t lds = (size_t)128 * (g.ldk + g.ldv) * 2;
    [[maybe_unused]] static const bool allowed = allow_lds((const void*)attn_stream_k<DH>, lds);
    const StreamMap map(a.F, a.skip, a.N, a.H, a.G);
    hipLaunchKernelGGL(attn_stream_k<DH>, dim3(map.grid), dim3(FW * 64), lds, s, a, map);
}

// ---- per-unit items ----------------------------------------------------------------------------
// A unit is one group of frames and one head.  The reference frame's keys are staged once; a
// non-reference frame reads each reused key from the reference's row and each recomputed key
// from its own row, through a per-frame key -> row map.  A frame's own rows, and those of
// consecutive frames, are consecutive packed rows (stable frame-major compaction; the reference
// frame is recomputed in full, its token i at packed row qoff[f0] + i), so staging is a copy of
// contiguous rows.  Every query tile of the unit goes to one wavefront, over all key blocks:
// no key split and no merge.
//
// LDS as UnitGeo lays it out.

// LDS rows dst0 .. dst0+count-1 of K and V <- packed rows src0 + min(i, nvalid - 1), head h
template <int DH, int NT>
__device__ __forceinline__ void stage_rows(const Geo& g, uint16_t* Ks, uint16_t* Vs,
                                           const uint16_t* qkv, size_t ld3, int D, int h, int dst0,
                                           int src0, int count, int nvalid, int tid) {
    constexpr int CH = DH / 8;
    const int total = count * CH;
    for (int c0 = tid; c0 < total; c0 += 4 * NT) {
        u32x4 kv[4], vv[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = min(c0 + u * NT, total - 1);
            const size_t off = (size_t)(src0 + min(c / CH, nvalid - 1)) * ld3 + h * DH + (c % CH) * 8;
            kv[u] = *(const u32x4*)(qkv + off + D);
            vv[u] = *(const u32x4*)(qkv + off + 2 * D);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + u * NT;
            if (c < total) {
                const int i = dst0 + c / CH, part = c % CH;
                *(u32x4*)(Ks + g.kofs(i, part)) = kv[u];
                *(u32x4*)(Vs + g.vofs(i, part)) = vv[u];
            }
        }
    }
}

template <int DH>
__global__ __launch_bounds__(UW * 64) __attribute__((amdgpu_waves_per_eu(3, 3)))
void attn_unit_k(AttnArgs a, int pcap) {
    constexpr int KS = DH / 16;
    constexpr int DB = (DH + 31) / 32;
    constexpr int NT = UW * 64;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int G = a.G, N = a.N, D = a.D, H = a.H;
    const UnitGeo ug(N, DH, G, pcap);
    const Geo& g = ug.g;
    uint16_t* Ks = (uint16_t*)smem;
    uint16_t* Vs = Ks + ug.vbase();
    uint16_t* kmap = Ks + ug.mbase();
    const uint16_t* qkv = (const uint16_t*)a.qkv;
    const size_t ld3 = 3 * (size_t)D;
    const int units = (a.F + G - 1) / G * H;
    const int Tref = (N + 31) / 32;   // query tiles of a reference frame
    for (int u = blockIdx.x; u < units; u += gridDim.x) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));   // keep lane-derived values inside the unit loop
        const int lane = tid & 63, wave = tid >> 6, hl = lane >> 5, lr = lane & 31;
        const int h = u % H, f0 = u / H * G, Gu = min(G, a.F - f0);
        const int r0 = a.qoff[f0];   // the reference frame's token i sits at packed row r0 + i
        stage_rows<DH, NT>(g, Ks, Vs, qkv, ld3, D, h, 0, r0, g.npad, N, tid);
        int Tr = Tref;               // reference tiles not taken yet
        int j = 1;
        do {
            // batch: frames j .. j2-1 of the group whose own rows fit in pcap (every frame's do:
            // pcap >= N), staged after the reference rows
            const int p0 = a.qoff[f0 + j];
            int j2 = j;
            while (j2 < Gu && a.qoff[f0 + j2 + 1] - p0 <= pcap) ++j2;
            const int prow = a.qoff[f0 + j2] - p0;
            if (prow > 0) stage_rows<DH, NT>(g, Ks, Vs, qkv, ld3, D, h, g.npad, p0, prow, prow, tid);
            for (int e = tid; e < (j2 - j) * g.npad; e += NT) {
                const int jj = j + e / g.npad, i = e % g.npad;
                const int p = a.pos[(size_t)(f0 + jj) * N + min(i, N - 1)];
                kmap[jj * g.npad + i] = (uint16_t)(p < r0 + N ? p - r0 : g.npad + p - p0);
            }
            lds_barrier();
            // the batch's tiles, then reference tiles: as many as fill the last round of
            // wavefronts, or all that are left after the last batch
            int Tb = 0;
            for (int jj = j; jj < j2; ++jj) Tb += (a.qoff[f0 + jj + 1] - a.qoff[f0 + jj] + 31) / 32;
            const int extra = j2 >= Gu ? Tr : min(Tr, (UW - Tb % UW) % UW);
            for (int t = wave; t < Tb + extra; t += UW) {
                int jj = -1, tt = t;   // frame (index in the group; -1: the reference) and tile
                if (t < Tb) {
                    jj = j;
                    for (int nt; tt >= (nt = (a.qoff[f0 + jj + 1] - a.qoff[f0 + jj] + 31) / 32); ++jj)
                        tt -= nt;
                } else {
                    tt = Tref - Tr + (t - Tb);
                }
                const int f = jj < 0 ? f0 : f0 + jj;
                const int q0 = a.qoff[f], q1 = a.qoff[f + 1];
                const int myq = q0 + tt * 32 + lr;
                const int qrow = myq < q1 ? myq : q1 - 1;
                bf16x8 qf[KS];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    qf[ks] = *(const bf16x8*)(qkv + (size_t)qrow * ld3 + h * DH + ks * 16 + hl * 8);
                float m, l;
                f32x16 o[DB];
                if (jj < 0) {
                    attend_tile<DH>(g, Ks, Vs, N, lane, qf, [](int k) { return k; }, m, l, o,
                                    [](int) {});
                } else {
                    const uint16_t* km = kmap + jj * g.npad;
                    attend_tile<DH>(g, Ks, Vs, N, lane, qf, [=](int k) { return (int)km[k]; },
                                    m, l, o, [](int) {});
                }
                if (myq < q1) store_row<DH>((uint16_t*)a.out + (size_t)myq * D + h * DH, lane, l, o);
            }
            Tr -= extra;
            lds_barrier();   // the next batch (or unit) restages rows and maps
            j = j2;
        } while (j < Gu);
    }
}

// ---- fp32 path ---------------------------------------------------------------------------------
// v_mfma_f32_16x16x4_f32 (fp32 products and sums), one query tile of 16 per wavefront, four
// wavefronts per block (frame, head, 64 queries).  The block stages 64 keys and values at a time in
// LDS (rows of dh + 4 floats: the fragment reads below hit distinct banks) and each wavefront takes
// one online-softmax step over them:
//   S^T = K . Q^T     lane l reads 16 bytes of key row l%16, dims 16 ks + 4 (l/16) + 0..3, the
//                     operands of four MFMAs; it ends with the scores of query l%16 for keys
//                     4 (l/16) + 0..3 of each block of 16
//   O^T += V^T . P^T  MFMA e takes keys 4 (l/16) + e: the probabilities as they sit, and V^T by
//                     4-byte reads
// A query's arithmetic depends on its frame's keys and values alone.  Bound by latency (staging,
// then one step after the other): scalar scores of a whole frame in one block per head took 853 us
// for 10 frames of 197 tokens, 12 heads, half of the queries active, and 71 us for 8 frames of 50
// tokens, 3 heads; this kernel 21.5 and 7.5 us.
constexpr int FK = 64;   // keys per step

template <int DT>   // dh / 16
__global__ __launch_bounds__(256) void attn_f32_k(AttnArgs a) {
    constexpr int DH = DT * 16, LD = DH + 4;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float* Ks = (float*)smem;
    float* Vs = Ks + FK * LD;
    const int f = blockIdx.x, h = blockIdx.y;
    const int q0 = a.qoff[f], q1 = a.qoff[f + 1];
    const int qb = q0 + (int)blockIdx.z * 64;
    if (qb >= q1) return;   // the whole block
    const int N = a.N, D = a.D;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, g = lane >> 4;
    const size_t ld3 = 3 * (size_t)D;
    const float* qkv = (const float*)a.qkv + (size_t)h * DH;
    const int myq = qb + wave * 16 + lr;
    const int qrow = myq < q1 ? myq : q1 - 1;   // tail lanes compute on a valid row
    const bool live = qb + wave * 16 < q1;      // wave-uniform
    const float scale = 1.0f / sqrtf((float)DH);
    f32x4 qf[DT], o[DT];
#pragma unroll
    for (int ks = 0; ks < DT; ++ks) {
        qf[ks] = *(const f32x4*)(qkv + (size_t)qrow * ld3 + ks * 16 + g * 4) * scale;
        o[ks] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float m = -INFINITY, l = 0.f;
    for (int k0 = 0; k0 < N; k0 += FK) {
        // keys past N repeat key N - 1 (finite data whose scores are masked)
#pragma unroll
        for (int u = 0; u < DT; ++u) {   // FK * DH / 4 pieces of each, 256 threads
            const int e = tid + u * 256, r = e / (DH / 4), c = e % (DH / 4);
            const size_t row = (size_t)a.pos[(size_t)f * N + min(k0 + r, N - 1)] * ld3 + c * 4;
            *(f32x4*)(Ks + r * LD + c * 4) = *(const f32x4*)(qkv + row + D);
            *(f32x4*)(Vs + r * LD + c * 4) = *(const f32x4*)(qkv + row + 2 * D);
        }
        __syncthreads();
        if (live) {
            const int nb = min(FK / 16, (N - k0 + 15) / 16);   // blocks of 16 with a key below N
            f32x4 sc[FK / 16];
            float mx = -INFINITY;
#pragma unroll
            for (int b = 0; b < FK / 16; ++b) {
                sc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (b < nb) {
#pragma unroll
                    for (int ks = 0; ks < DT; ++ks) {
                        const f32x4 kf = *(const f32x4*)(Ks + (b * 16 + lr) * LD + ks * 16 + g * 4);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            sc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[e], qf[ks][e], sc[b], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (k0 + b * 16 + g * 4 + e >= N) sc[b][e] = -INFINITY;
                    mx = fmaxf(mx, sc[b][e]);
                }
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            const float mn = fmaxf(m, mx);
            const float alpha = expf(m - mn);   // 0 at the first step
            float ps = 0.f;
#pragma unroll
            for (int b = 0; b < FK / 16; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sc[b][e] = expf(sc[b][e] - mn);
                    ps += sc[b][e];
                }
            ps += __shfl_xor(ps, 16, 64);
            ps += __shfl_xor(ps, 32, 64);
            l = l * alpha + ps;
            m = mn;
#pragma unroll
            for (int d = 0; d < DT; ++d) o[d] *= alpha;
#pragma unroll
            for (int b = 0; b < FK / 16; ++b) {
                if (b >= nb) break;
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int d = 0; d < DT; ++d)
                        o[d] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            Vs[(b * 16 + g * 4 + e) * LD + d * 16 + lr], sc[b][e], o[d], 0, 0, 0);
            }
        }
        __syncthreads();   // the next step restages the keys and values
    }
    if (myq >= q1) return;
    float* dst = (float*)a.out + (size_t)myq * D + (size_t)h * DH;
#pragma unroll
    for (int d = 0; d < DT; ++d) *(f32x4*)(dst + d * 16 + g * 4) = o[d] * (1.0f / l);
}

template <int DT>
void launch_f32(const AttnArgs& a, hipStream_t s) {
    constexpr size_t lds = (size_t)2 * FK * (DT * 16 + 4) * sizeof(float);
    [[maybe_unused]] static const bool allowed = allow_lds((const void*)attn_f32_k<DT>, lds);
    hipLaunchKernelGGL(attn_f32_k<DT>, dim3(a.F, a.H, (a.N + 63) / 64), dim3(256), lds, s, a);
}

// ---- class-token attention weights (the decision MLP's importance cue) ------------------------
// One wavefront per (non-reference frame, head): the class query's scores against the frame's N
// keys (read through pos), then their softmax.  Eight lanes share a key: each multiplies one or
// more 16-byte chunks of the key row with the matching chunks of the query (held in registers),
// so a wavefront reads eight key rows per step in whole 128-byte segments; the eight partial
// sums meet in three shuffles.  Four heads per block, no block barriers (each wavefront has its
// own LDS slice).
template <bool BF>
__device__ inline float elem_at(const void* p, size_t i) {
    if constexpr (BF) return bf16_to_f32(((const uint16_t*)p)[i]);
    else return ((const float*)p)[i];
}

template <bool BF>
__global__ __launch_bounds__(256) void cls_attn_k(AttnArgs a, float* __restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int CE = BF ? 8 : 4;            // elements per 16-byte chunk
    constexpr int U = 128 / CE / 8;           // chunks per lane for a head dim of up to 128
    constexpr int KB = 4;                     // steps of eight keys whose loads are in flight together
    const int f = blockIdx.x;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int h = blockIdx.y * 4 + wave;
    // reference frames are never gated; frames carried over from an earlier call have no rows
    if ((a.G > 0 && f % a.G == 0) || f < a.skip || h >= a.H) return;
    const int N = a.N, D = a.D, dh = D / a.H, nch = dh / CE;
    const int sub = lane & 7, kq = lane >> 3;
    float* sc = (float*)smem + (size_t)wave * N;   // scores, then exponentials
    const size_t ld3 = 3 * (size_t)D;
    const size_t qrow = (size_t)a.qoff[f] * ld3 + (size_t)h * dh;   // the frame's first row
    float q[U][CE];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < CE; ++e) {
            const int c = sub + 8 * u;
            q[u][e] = c < nch ? elem_at<BF>(a.qkv, qrow + (size_t)c * CE + e) : 0.f;
        }
    const float scale = 1.0f / sqrtf((float)dh);
    typedef typename std::conditional<BF, uint4, float4>::type chunk_t;
    // key rows' packed indices of the steps at j0, loaded one iteration ahead so that an
    // iteration waits for one memory round trip (the key rows), not two
    int pr[KB];
    auto rows_at = [&](int j0, int (&dst)[KB]) {
#pragma unroll
        for (int t = 0; t < KB; ++t) {
            const int j = j0 + 8 * t + kq;
            dst[t] = j < N ? a.pos[(size_t)f * N + j] : 0;
        }
    };
    rows_at(0, pr);
    for (int j0 = 0; j0 < N; j0 += 8 * KB) {
        // KB steps of eight keys at once: every row offset, then every chunk, then the sums
        size_t kr[KB];
#pragma unroll
        for (int t = 0; t < KB; ++t) {
            const int j = j0 + 8 * t + kq;
            kr[t] = j < N ? (size_t)pr[t] * ld3 + D + (size_t)h * dh : 0;
        }
        if (j0 + 8 * KB < N) rows_at(j0 + 8 * KB, pr);
        chunk_t kv[KB][U];
#pragma unroll
        for (int t = 0; t < KB; ++t)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = sub + 8 * u, j = j0 + 8 * t + kq;
                if (j < N && c < nch) {
                    kv[t][u] = *(const chunk_t*)((const char*)a.qkv +
                                                 (kr[t] + (size_t)c * CE) * (BF ? 2 : 4));
                } else {
                    kv[t][u] = chunk_t{0, 0, 0, 0};
                }
            }
#pragma unroll
        for (int t = 0; t < KB; ++t) {
            float s = 0.f;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if constexpr (BF) {
                    const uint32_t w[4] = {kv[t][u].x, kv[t][u].y, kv[t][u].z, kv[t][u].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        s = fmaf(q[u][2 * e], bf16_to_f32((uint16_t)(w[e] & 0xFFFFu)), s);
                        s = fmaf(q[u][2 * e + 1], bf16_to_f32((uint16_t)(w[e] >> 16)), s);
                    }
                } else {
                    s = fmaf(q[u][0], kv[t][u].x, s);
                    s = fmaf(q[u][1], kv[t][u].y, s);
                    s = fmaf(q[u][2], kv[t][u].z, s);
                    s = fmaf(q[u][3], kv[t][u].w, s);
                }
            }
            s += __shfl_xor(s, 1, 64);
            s += __shfl_xor(s, 2, 64);
            s += __shfl_xor(s, 4, 64);
            const int j = j0 + 8 * t + kq;
            if (sub == 0 && j < N) sc[j] = s * scale;
        }
    }
    wave_lds_sync();
    float mx = -INFINITY;
    for (int j = lane; j < N; j += 64) mx = fmaxf(mx, sc[j]);
    mx = wmax(mx);
    float sum = 0.f;
    for (int j = lane; j < N; j += 64) {
        const float e = expf(sc[j] - mx);
        sc[j] = e;
        sum += e;
    }
    const float inv = 1.0f / wsum(sum);
    float* o = out + ((size_t)f * a.H + h) * N;
    for (int j = lane; j < N; j += 64) o[j] = sc[j] * inv;
}

// The fp32 token counts accepted: a head's keys, values, four queries and their scores in LDS (the
// kernel stages 64 keys at a time and needs less).
size_t f32_lds_bytes(int N, int dh) {
    return ((size_t)N * (dh + 1) + (size_t)N * dh + (size_t)4 * dh + (size_t)4 * N) * 4;
}

template <int DH>
void launch_bf16(const AttnArgs& a, hipStream_t s) {
    const AttnPlan p = attn_plan<DH>(a);
    if constexpr (DH == 64) {
        [[maybe_unused]] static const bool allowed = allow_lds((const void*)attn_unit_k<DH>, ATTN_LDS);
        if (p.route == ATTN_UNIT)
            hipLaunchKernelGGL(attn_unit_k<DH>, dim3(p.grid), dim3(UW * 64), p.lds, s, a, p.pcap);
    }
    if constexpr (frame_blocks(DH) > 0) {
        [[maybe_unused]] static const bool allowed = allow_lds((const void*)attn_mfma_k<DH>, ATTN_LDS);
        if (p.route == ATTN_FRAME)
            hipLaunchKernelGGL(attn_mfma_k<DH>, dim3(p.grid), dim3(AW * 64), p.lds, s, a);
    }
    if (p.route == ATTN_STREAM) launch_stream<DH>(a, s);
}

}  // namespace

size_t attention_lds_bytes(bool bf16, int N, int dh) {
    return bf16 ? Geo(N, dh).bytes() : f32_lds_bytes(N, dh);
}

bool attention_supported(bool bf16, int N, int dh) {
    if (attention_lds_bytes(bf16, N, dh) > ATTN_LDS) return false;
    if (bf16) return dh == 64 || dh == 80 || dh == 96 || dh == 128;
    return dh % 16 == 0;
}

void launch_cls_attention(bool bf16, const AttnArgs& a, float* probs, hipStream_t s) {
    const size_t lds = 4 * (size_t)a.N * sizeof(float);
    const dim3 grid(a.F, (a.H + 3) / 4);
    if (bf16) hipLaunchKernelGGL(cls_attn_k<true>, grid, dim3(256), lds, s, a, probs);
    else hipLaunchKernelGGL(cls_attn_k<false>, grid, dim3(256), lds, s, a, probs);
}

void launch_attention(bool bf16, const AttnArgs& a, hipStream_t s) {
    const int dh = a.D / a.H;
    if (!bf16) {
        switch (dh / 16) {
            case 1: launch_f32<1>(a, s); break;
            case 2: launch_f32<2>(a, s); break;
            case 3: launch_f32<3>(a, s); break;
            case 4: launch_f32<4>(a, s); break;
            case 5: launch_f32<5>(a, s); break;
            case 6: launch_f32<6>(a, s); break;
            case 7: launch_f32<7>(a, s); break;
            case 8: launch_f32<8>(a, s); break;
            default: break;  // rejected at handle creation
        }
        return;
    }
    switch (dh) {
        case 64: launch_bf16<64>(a, s); break;
        case 80: launch_bf16<80>(a, s); break;
        case 96: launch_bf16<96>(a, s); break;
        case 128: launch_bf16<128>(a, s); break;
        default: break;  // rejected at handle creation
    }
}

}  // namespace dv
