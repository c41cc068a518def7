// Packed-row GEMMs: C[M, Nout] = A[M, K] * W[Nout, K]^T + fused epilogue.
//
// M (the number of packed recompute rows) lives in device memory; a workgroup per compute unit (fp32:
// two) walks the live tiles, fewer where the largest possible M has fewer tiles, and one without a
// tile returns at once.
//
// bf16 path: MFMA v_mfma_f32_32x32x16_bf16 with fp32 accumulation.
//   * One workgroup of eight wavefronts per compute unit walks block tiles BM x BN; the wavefronts
//     share a tile WGM x WGN, each owning (BM/WGM) x (BN/WGN) of 32 x 32 tiles.
//   * Whole rounds of the grid take 256 x 256 tiles (256 x 128 where Nout is no multiple of 256);
//     the rows left over take the tile shape that finishes them soonest (gemm_plan).
//   * k-slices of 64 travel global -> LDS with buffer_load_dwordx4 ... lds (no staging registers)
//     through a ring of S stages.  One wavefront instruction writes 1 KiB of LDS (lane i at
//     base + 16 i).  LDS rows are 128 bytes without padding; lane i fetches the global chunk that
//     belongs at its slot: chunk c of tile row r sits at slot c ^ swz(r), so 16 lanes reading one
//     chunk of 16 rows hit distinct banks.
//   * Both operands are K-contiguous rows, so A and B fragments are the same 16-byte LDS read:
//     lane l takes row l%32 and k-slice (l/32)*8 .. +8.  The weight fragment is the MFMA's
//     first operand, so the accumulator is the transposed tile: lane l, register j holds output
//     column (j/4)*8 + (l/32)*4 + j%4 of token row l%32 -- four consecutive columns per
//     register group, stored as one vector by the epilogue.
//   * The fragments of k-step ks+1 are read while the MFMAs of k-step ks run; the smallest tiles
//     read a whole slice ahead (one MFMA per k-step does not cover an LDS read).
//   * Tile order: the live tiles (ceil(M/BM) * Nout/BN) go round-robin over the 8 XCDs in
//     contiguous chunks, each chunk walking groups of 8 tile-rows across all tile-columns, so
//     an XCD's L2 sees few distinct A and W tiles.
//   * Every output is one chain of MFMAs in k order from its bias, whatever tile takes it, so a
//     row's result does not depend on how many other rows the launch has.
//
// fp32 path: the same scheme on v_mfma_f32_16x16x4_f32 (f32_tile).
#include <algorithm>
#include <type_traits>

#include "dv_internal.h"

namespace dv {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

__device__ inline float gelu_erf(float v) { return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f)); }

// GELU for outputs rounded to bf16: with y = x clamped to [-4, 4], Phi(x) = 1/2 + y P(y^2), P a
// degree-8 least-squares fit to the normal CDF on [0, 4] with 4 P(16) = 1/2 imposed
// (coefficients from gelu_fit.py), so that past |x| = 4 the result is x or 0.  GELU = x Phi(x):
// 12 VALU operations, no transcendental.  |GELU error| <= 1.1e-5 for |x| <= 3 and <= 1.3e-4
// everywhere (largest near |x| = 4): far below the bf16 step (2^-8 relative) of the result.
__device__ inline float gelu_poly(float x) {
    const float y = __builtin_amdgcn_fmed3f(x, -4.0f, 4.0f);
    const float s = y * y;
    float p = 9.151786967e-11f;
    p = fmaf(p, s, -7.699238580e-09f);
    p = fmaf(p, s, 2.898779599e-07f);
    p = fmaf(p, s, -6.548660622e-06f);
    p = fmaf(p, s, 1.009105545e-04f);
    p = fmaf(p, s, -1.142885303e-03f);
    p = fmaf(p, s, 9.898823686e-03f);
    p = fmaf(p, s, -6.643372774e-02f);
    p = fmaf(p, s, 3.989303410e-01f);
    return x * fmaf(y, p, 0.5f);
}

__device__ inline u32x2 pack_bf16x4(f32x4 v) {
    bf16x4 h = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};  // v_cvt_pk_bf16_f32 (RNE)
    return __builtin_bit_cast(u32x2, h);
}

// fp32 path: the sums (bias included) of four consecutive columns of one row to their output
template <Epi E>
__device__ inline void epi_store4(const GemmArgs& a, int row, int col, f32x4 v) {
    auto at = [&](const float* p, size_t r) { return *(const f32x4*)(p + r * a.Nout + col); };
    size_t o = row;   // output row
    if constexpr (E == Epi::Patch) {
        const int f = row / a.P, k = row - f * a.P;
        v += at(a.pos, 1 + k);
        o = (size_t)f * a.N + 1 + k;
    } else if constexpr (E == Epi::OProj) {
        v += at(a.resid, a.idx[row]);
    } else if constexpr (E == Epi::Fc1) {
        v = f32x4{gelu_erf(v[0]), gelu_erf(v[1]), gelu_erf(v[2]), gelu_erf(v[3])};
    } else if constexpr (E == Epi::Fc2) {
        v += at(a.resid, row);
        o = a.idx[row];
    } else if constexpr (E == Epi::Restore) {   // a reused token's row from its reference's new row
        const int t = a.idx[row], f = t / a.N;
        v += at(a.resid, (size_t)(f / a.G * a.G) * a.N + t % a.N);
        o = t;
    }
    *(f32x4*)((float*)a.out + o * a.Nout + col) = v;
}

__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Buffer descriptor over `bytes` bytes at p (raw, no stride): a load or store whose 32-bit byte
// offset falls past `bytes` is dropped by the hardware range check.  Every workspace buffer is below
// 2^32 bytes (rows, padding included, are checked at handle creation), so offsets into it are plain
// 32-bit products and need no 64-bit address arithmetic; weights are addressed from their tile.
__device__ inline __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
constexpr uint32_t out_bytes(Epi e) { return e == Epi::Qkv || e == Epi::Fc1 ? 2 : 4; }   // per element

// Epilogue of one wavefront's (TI*32) x (TJ*32) sub-tile, staged through a wave-private LDS
// slab so that global traffic is row-contiguous: for each 32-row slab the accumulators (lane l
// holds row l%32, columns (r/4)*8 + (l/32)*4 + r%4 of each 32-column tile) are written to LDS,
// then read back row-major -- each lane owns 4 fixed columns, and a wavefront instruction covers
// 64/(TJ*8) whole row segments.  The accumulators already hold the bias.  Row indices of every
// slab are requested up front and the residual (or position) rows of slab i+1 are in flight
// while slab i is combined and stored.  Stores go through buffer descriptors: rows past M in
// the tile tail get an offset past the descriptor and are dropped.  The caller has finished
// with the LDS ring.
template <Epi E, int TI, int TJ>
__device__ inline void epilogue_lds(const GemmArgs& a, f32x16 (&acc)[TI][TJ], float* slab, int row0,
                                    int col0, int M, int lane) {
    constexpr int WN = TJ * 32;          // columns of the sub-tile
    constexpr int LDW = WN + 4;          // padded slab row (floats)
    constexpr int CPRW = WN / 4;         // 16-byte chunks per row
    constexpr int RPI = 64 / CPRW;       // rows per wavefront instruction
    constexpr int NQ = 32 / RPI;         // instructions per 32-row slab
    constexpr bool LOADS = E == Epi::OProj || E == Epi::Fc2 || E == Epi::Patch || E == Epi::Restore;
    // output rows are token rows
    constexpr bool SCATTER = E == Epi::Fc2 || E == Epi::Patch || E == Epi::Restore;
    constexpr uint32_t ESZ = out_bytes(E);
    const int lr = lane & 31, hl = lane >> 5;
    const int c = lane % CPRW, rsub = lane / CPRW;
    const uint32_t col = col0 + c * 4;
    const uint32_t Nout = a.Nout;
    // packed-row outputs end at row M; token-row outputs drop tail rows by their offset
    const auto rout = buf_rsrc(a.out, SCATTER ? BUF_ANY : (uint32_t)M * Nout * ESZ);
    const auto rres = buf_rsrc(E == Epi::Patch ? (const void*)a.pos : (const void*)a.resid, BUF_ANY);

    auto row_of = [&](int i, int q) { return row0 + i * 32 + q * RPI + rsub; };
    // residual (or position) rows and output offsets of slab i; one slab ahead
    f32x4 extra[2][NQ];
    uint32_t ooff[2][NQ];
    auto fetch = [&](int i, f32x4 (&dst)[NQ], uint32_t (&oo)[NQ]) {
        int tr[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int row = row_of(i, q);
            const int r = row < M ? row : M - 1;           // a valid row for the tile tail
            if constexpr (E == Epi::OProj || E == Epi::Fc2 || E == Epi::Restore) tr[q] = a.idx[r];
            else if constexpr (E == Epi::Patch) tr[q] = (r / a.P) * a.N + 1 + r % a.P;
            else tr[q] = row;
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int row = row_of(i, q);
            if constexpr (SCATTER)
                oo[q] = row < M ? ((uint32_t)tr[q] * Nout + col) * ESZ : BUF_ANY;
            else
                oo[q] = ((uint32_t)row * Nout + col) * ESZ;   // past M: past the records (gemm_plan)
        }
        if constexpr (LOADS) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int row = row_of(i, q);
                const uint32_t r = row < M ? row : M - 1;
                uint32_t off;
                if constexpr (E == Epi::OProj) {
                    off = ((uint32_t)tr[q] * Nout + col) * 4;
                } else if constexpr (E == Epi::Fc2) {
                    off = (r * Nout + col) * 4;
                } else if constexpr (E == Epi::Restore) {   // the reference token's row
                    const uint32_t t = tr[q], f = t / a.N;
                    off = (((f / a.G * a.G) * a.N + t % a.N) * Nout + col) * 4;
                } else {
                    off = ((1 + r % a.P) * Nout + col) * 4;
                }
                dst[q] = __builtin_amdgcn_raw_buffer_load_b128(rres, (int)off, 0, 0);
            }
        }
    };
    fetch(0, extra[0], ooff[0]);
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        if (i + 1 < TI) fetch(i + 1, extra[(i + 1) & 1], ooff[(i + 1) & 1]);
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 v = {acc[i][j][g * 4 + 0], acc[i][j][g * 4 + 1], acc[i][j][g * 4 + 2],
                           acc[i][j][g * 4 + 3]};
                *(f32x4*)(slab + lr * LDW + j * 32 + g * 8 + hl * 4) = v;
            }
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int r = q * RPI + rsub;
            const f32x4 v = *(const f32x4*)(slab + r * LDW + c * 4);   // bias included
            const int off = (int)ooff[i & 1][q];
            if constexpr (E == Epi::Qkv) {
                __builtin_amdgcn_raw_buffer_store_b64(pack_bf16x4(v), rout, off, 0, 0);
            } else if constexpr (E == Epi::Fc1) {
                const f32x4 gl = {gelu_poly(v[0]), gelu_poly(v[1]), gelu_poly(v[2]), gelu_poly(v[3])};
                __builtin_amdgcn_raw_buffer_store_b64(pack_bf16x4(gl), rout, off, 0, 0);
            } else if constexpr (E == Epi::Delta) {
                __builtin_amdgcn_raw_buffer_store_b128(v, rout, off, 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b128(v + extra[i & 1][q], rout, off, 0, 0);
            }
        }
        wave_lds_sync();   // the slab is rewritten by the next 32-row slab
    }
}

// s_waitcnt vmcnt(n) lgkmcnt(0) (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4 left
// at its maximum, lgkmcnt 11:8): all of this wave's loads but the last n have landed in LDS and
// its own LDS reads are complete.
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14));
}

// Workgroup barrier without the memory fence of __syncthreads() (that fence would wait for
// every load in flight, i.e. drain the LDS ring).  Callers order memory with wait_vm first; the
// signal fences stop the compiler from moving memory accesses across the barrier.
__device__ __forceinline__ void bare_barrier() {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_barrier();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Tile of launch index bid among mt x tilesN live tiles: the tiles go round-robin over the 8 XCDs
// in contiguous chunks, each chunk walking groups of 8 tile-rows across all tile-columns, so an
// XCD's L2 sees few distinct A and W tiles at a time.
__device__ __forceinline__ void tile_coords(int bid, int mt, int tilesN, int& tm, int& tn) {
    const int active = mt * tilesN;
    int lid = bid;
    const int per = active / 8;
    if (bid < per * 8) lid = (bid % 8) * per + bid / 8;
    constexpr int GM = 8;
    const int group = lid / (GM * tilesN);
    const int first_m = group * GM;
    const int gsize = min(mt - first_m, GM);
    const int w_in = lid - group * GM * tilesN;
    tn = gsize == GM ? w_in / GM : w_in / gsize;   // all groups but the last: a shift
    tm = first_m + w_in - tn * gsize;
}

// f(R), f(R - 1), ..., f(1) with compile-time arguments
template <int R, class F>
__device__ __forceinline__ void drain(F f) {
    if constexpr (R > 0) {
        f(std::integral_constant<int, R>());
        drain<R - 1>(f);
    }
}

// ---------------- bf16 MFMA GEMM, pipelined ----------------------------------------------------
// One block tile: the DMA ring keeps S-1 k-slices in flight and the MFMA fragments are always one
// k-step ahead, across stage boundaries too.  The barrier of stage kt+1 sits just before the first
// fragment loads of stage kt+1; the DMA of a new stage is issued right after it, into the slot
// every wave finished reading before that barrier.  The tile is number `bid` of the rows [m0, M);
// `sm` is the workgroup's LDS.  Every wavefront of the workgroup passes the same barriers.
// AHEAD (tiles whose wavefronts have one MFMA per k-step): the fragments of a whole slice are read
// one slice ahead, so a slice costs one barrier and one LDS latency instead of one per k-step, and
// S slices are in flight.
// PERSIST: the block goes on to tiles bid + stride, bid + 2 stride, ... of the same rows; when a
// tile's last k-slice starts, the next tile's first slice and bias are copied into the ring slot
// that is then free (an even number of slices; else between the tiles), and the epilogue's slabs
// sit past that slot.
template <Epi E, int BM, int BN, int BKD, int S, int WGM, int WGN, bool PERSIST = false,
          bool AHEAD = false>
__device__ __forceinline__ void pipe_tile(const GemmArgs& a, uint16_t* sm, int bid, int m0, int M,
                                          int wave, int stride = 0) {
    constexpr int NW = WGM * WGN;                 // wavefronts, WGM x WGN over the block tile
    constexpr int WM = BM / WGM, WN = BN / WGN, TI = WM / 32, TJ = WN / 32;
    constexpr int CPR = BKD / 8;
    constexpr int RPI = 64 / CPR;
    constexpr int SH = (CPR == 8) ? 1 : 2;
    constexpr int LA = BM / RPI / NW, LB = BN / RPI / NW;
    static_assert(LA * RPI * NW == BM && LB * RPI * NW == BN, "load split");
    constexpr int L = LA + LB;
    constexpr int STAGE = (BM + BN) * BKD;
    constexpr int KS = BKD / 16;
    static_assert(KS % 2 == 0, "fragment double buffer assumes an even number of k-steps");

    const int tilesN = a.Nout / BN;
    const int mt = (M - m0 + BM - 1) / BM;
    const int active = mt * tilesN;
    if (bid >= active) return;
    int tm, tn;

    const int lane = threadIdx.x & 63;
    const int wm = wave / WGN, wn = wave % WGN;
    const int lr = lane & 31, hl = lane >> 5;
    const int K = a.K;

    // this lane's DMA chunks: 32-bit byte offsets into the A buffer (below 2^32 bytes) and the tile's
    // own weight rows (a weight matrix may be larger); the k-slice advance rides in the scalar
    // offset of buffer_load ... lds
    const int lrow = lane / CPR, lslot = lane % CPR;
    uint32_t goffA[LA], goffB[LB];
    __amdgpu_buffer_rsrc_t rW;
    auto setup = [&](int b, int& tm_, int& tn_) {
        tile_coords(b, mt, tilesN, tm_, tn_);
#pragma unroll
        for (int t = 0; t < LA; ++t) {
            const int r = (wave * LA + t) * RPI + lrow;
            const int c = lslot ^ ((r >> SH) & (CPR - 1));
            const int grow = m0 + tm_ * BM + r;
            const int live = grow < M ? grow : M - 1;   // rows past M repeat the last one
            const int arow = a.a_idx ? a.a_idx[live] : live;   // gathered A rows
            goffA[t] = ((uint32_t)arow * K + c * 8) * 2;
        }
#pragma unroll
        for (int t = 0; t < LB; ++t) {
            const int r = (wave * LB + t) * RPI + lrow;
            const int c = lslot ^ ((r >> SH) & (CPR - 1));
            goffB[t] = ((uint32_t)r * K + c * 8) * 2;
        }
        rW = buf_rsrc((const char*)a.W + (uint64_t)(uint32_t)(tn_ * BN) * (uint32_t)(K * 2), BUF_ANY);
    };
    setup(bid, tm, tn);
    const auto rA = buf_rsrc(a.A, BUF_ANY);
    const auto rBias = buf_rsrc(a.bias, BUF_ANY);
    // copy t of slice kt (weights first) into ring slot `slot`.  Slots are counted along with the
    // slices: a division by a ring depth that is no power of two costs more than a k-step's MFMA.
    auto load1 = [&](int slot, int kt, int t) {
        uint16_t* st = sm + slot * STAGE;
        const int soff = kt * BKD * 2;
        if (t < LB)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rW,
                (__attribute__((address_space(3))) void*)(st + BM * BKD + (wave * LB + t) * RPI * BKD), 16,
                (int)goffB[t < LB ? t : 0], soff, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rA,
                (__attribute__((address_space(3))) void*)(st + (wave * LA + t - LB) * RPI * BKD), 16,
                (int)goffA[t < LB ? 0 : t - LB], soff, 0, 0);
    };
    auto issue = [&](int slot, int kt) {
#pragma unroll
        for (int t = 0; t < L; ++t) load1(slot, kt, t);
    };
    auto after = [](int slot) { return slot + 1 == S ? 0 : slot + 1; };
    // persistent tiles: the tile's bias (BN floats) goes to LDS past the slabs with the DMA of its
    // first slice, so that setting the accumulators waits on no vector memory operation (a
    // global load there would also wait for the previous epilogue's stores)
    constexpr size_t RING_B = (size_t)S * STAGE * 2;
    constexpr size_t SLAB_END = (size_t)STAGE * 2 + (size_t)NW * 32 * (TJ * 32 + 4) * 4;
    float* const bias_lds = (float*)((char*)sm + (RING_B > SLAB_END ? RING_B : SLAB_END));
    auto issue_bias = [&](int tn_) {
        if constexpr (PERSIST) {
            static_assert(BN % 64 == 0 && BN / 64 <= NW, "one 64-float piece per wavefront");
            if (wave < BN / 64)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rBias,
                    (__attribute__((address_space(3))) void*)(bias_lds + wave * 64), 4,
                    (int)((tn_ * BN + wave * 64 + lane) * 4), 0, 0, 0);
        }
    };
    // per-lane LDS element offsets of the fragments (row part; the chunk is XORed per k-step)
    int offA[TI], offB[TJ], swA[TI], swB[TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i) {
        const int r = wm * WM + i * 32 + lr;
        offA[i] = r * BKD;
        swA[i] = (r >> SH) & (CPR - 1);
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
        const int r = wn * WN + j * 32 + lr;
        offB[j] = BM * BKD + r * BKD;
        swB[j] = (r >> SH) & (CPR - 1);
    }
    auto frag = [&](int slot, int ks, bf16x8 (&xa)[TI], bf16x8 (&xb)[TJ]) {
        const uint16_t* st = sm + slot * STAGE;
        const int c = ks * 2 + hl;
        // in the order the products need them (B0, A0, B1, ...)
#pragma unroll
        for (int q = 0; q < TI + TJ; ++q) {
            const int n = q < 2 * TJ ? q / 2 : q - TJ;
            if (q < 2 * TJ && q % 2 == 0) xb[n] = *(const bf16x8*)(st + offB[n] + (c ^ swB[n]) * 8);
            else if (n < TI) xa[n] = *(const bf16x8*)(st + offA[n] + (c ^ swA[n]) * 8);
        }
    };

    f32x16 acc[TI][TJ];
    const int nk = K / BKD;
    f32x4 bias_r[TJ][4];   // one tile per call: the bias is requested ahead of the ring
    if constexpr (!PERSIST) {
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                bias_r[j][g] = *(const f32x4*)(a.bias + tn * BN + wn * WN + j * 32 + g * 8 + hl * 4);
    }
#pragma unroll
    for (int p = 0; p < (AHEAD ? S : S - 1); ++p)
        if (p < nk) issue(p, p);
    issue_bias(tn);
    if (PERSIST || nk < (AHEAD ? S : S - 1)) wait_vm<0>();
    else wait_vm<(AHEAD ? S - 1 : S - 2) * L>();   // the first slice has landed
    bare_barrier();
    bf16x8 fa[2][TI], fb[2][TJ];
    // one k-slice: MFMAs on the fragments in hand while the next fragments are read.  NEXT:
    // whether the following slice's first fragments are read at the end (after its barrier);
    // WAITN: vmcnt that guarantees the following slice has landed.  The three uses below are
    // separate instantiations, so the steady-state loop body has no branch.
    auto mfmas = [&](int cur, int from, int to) {
#pragma unroll
        for (int q = from; q < to; ++q) {
            const int i = q / TJ, j = q % TJ;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cur][j], fa[cur][i], acc[i][j],
                                                                0, 0, 0);
        }
    };
    // Interleave for one k-step (in-order issue: a read placed after a run of MFMAs would wait
    // for the MFMA pipe): reads of the next fragments go between the MFMAs of this k-step.
    constexpr int NM = TI * TJ, NR = TI + TJ;      // MFMAs and fragment reads per k-step
    constexpr int PAIRS = NR < NM ? NR : NM;
    constexpr int PRE = NM / 4;                    // MFMAs issued before a stage barrier
    constexpr int PAIRS2 = NR < NM - PRE ? NR : NM - PRE;
    int slot = 0;   // of the slice at hand
    auto slice = [&](int kt, auto next, auto waitn) {
        if constexpr (S == 2) slot = kt & 1;
        const int nslot = S == 2 ? (kt + 1) & 1 : after(slot);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int cur = ks & 1;
            if (ks + 1 < KS) {
                frag(slot, ks + 1, fa[cur ^ 1], fb[cur ^ 1]);
                mfmas(cur, 0, NM);
#pragma unroll
                for (int q = 0; q < PAIRS; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
                }
                if constexpr (NR > PAIRS) __builtin_amdgcn_sched_group_barrier(0x100, NR - PAIRS, 0);
                if constexpr (NM > PAIRS) __builtin_amdgcn_sched_group_barrier(0x008, NM - PAIRS, 0);
                __builtin_amdgcn_sched_barrier(0);
            } else if constexpr (decltype(next)::value) {
                mfmas(cur, 0, PRE);
                __builtin_amdgcn_sched_barrier(0);
                wait_vm<decltype(waitn)::value>();
                bare_barrier();
                frag(nslot, 0, fa[cur ^ 1], fb[cur ^ 1]);
                mfmas(cur, PRE, NM);
#pragma unroll
                for (int q = 0; q < PAIRS2; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                }
                if constexpr (NR > PAIRS2) __builtin_amdgcn_sched_group_barrier(0x100, NR - PAIRS2, 0);
                if constexpr (NM - PRE > PAIRS2) __builtin_amdgcn_sched_group_barrier(0x008, NM - PRE - PAIRS2, 0);
                __builtin_amdgcn_sched_barrier(0);
            } else {
                mfmas(cur, 0, NM);
            }
        }
        slot = nslot;
    };
    using T_ = std::integral_constant<bool, true>;
    using F_ = std::integral_constant<bool, false>;
    for (;;) {   // one tile; persistent head blocks go on to tile bid + stride
        slot = 0;
        // the accumulators start at the bias of their column (lane l, register r of MFMA tile j:
        // column (r/4)*8 + (l/32)*4 + r%4 of the tile), so the epilogue does not add it
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
            f32x16 b;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int bc = wn * WN + j * 32 + g * 8 + hl * 4;
                f32x4 v;
                if constexpr (PERSIST) v = *(const f32x4*)(bias_lds + bc);
                else v = bias_r[j][g];
#pragma unroll
                for (int e = 0; e < 4; ++e) b[g * 4 + e] = v[e];
            }
#pragma unroll
            for (int i = 0; i < TI; ++i) acc[i][j] = b;
        }

        int kt = 0;
        if constexpr (AHEAD) {
            bf16x8 ga[2][KS][TI], gb[2][KS][TJ];
            auto read_slice = [&](int sl, bf16x8 (&xa)[KS][TI], bf16x8 (&xb)[KS][TJ]) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) frag(sl, ks, xa[ks], xb[ks]);
            };
            // the MFMAs of a slice are one chain: the copies of slice kl go between them
            auto mul_slice = [&](const bf16x8 (&xa)[KS][TI], const bf16x8 (&xb)[KS][TJ], int kl, auto load) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                    for (int q = 0; q < TI * TJ; ++q) {
                        const int i = q / TJ, j = q % TJ;
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xb[ks][j], xa[ks][i],
                                                                            acc[i][j], 0, 0, 0);
                    }
                    if constexpr (decltype(load)::value) {
#pragma unroll
                        for (int t = ks; t < L; t += KS) load1(slot, kl, t);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            auto step = [&](int k, auto waitn, auto load, auto par) {
                constexpr int P = decltype(par)::value;
                wait_vm<decltype(waitn)::value>();
                bare_barrier();
                const int nslot = after(slot);
                read_slice(nslot, ga[P ^ 1], gb[P ^ 1]);
                __builtin_amdgcn_sched_barrier(0);
                mul_slice(ga[P], gb[P], k + S, load);   // slice k + S takes the slot of slice k
                __builtin_amdgcn_sched_barrier(0);
                slot = nslot;
            };
            using P0 = std::integral_constant<int, 0>; using P1 = std::integral_constant<int, 1>;
            using W = std::integral_constant<int, (S - 2) * L>;
            read_slice(0, ga[0], gb[0]);
            for (; kt + 1 + S < nk; kt += 2) {
                step(kt, W(), T_(), P0());
                step(kt + 1, W(), T_(), P1());
            }
            if (kt + S < nk) {
                step(kt, W(), T_(), P0());
                ++kt;
            }
            drain<S - 1>([&](auto r) {
                constexpr int R = decltype(r)::value;
                if (nk - 1 - kt >= R) {
                    using WR = std::integral_constant<int, (R - 1) * L>;
                    if (kt & 1) step(kt, WR(), F_(), P1());
                    else step(kt, WR(), F_(), P0());
                    ++kt;
                }
            });
            if (kt & 1) mul_slice(ga[1], gb[1], 0, F_());
            else mul_slice(ga[0], gb[0], 0, F_());
        } else {
            frag(0, 0, fa[0], fb[0]);
            for (; kt + S - 1 < nk; ++kt) {   // steady state: a new slice enters the ring every step
                // into the slot of slice kt-1: every wave read it before a barrier
                issue(S == 2 ? (kt + 1) & 1 : slot == 0 ? S - 1 : slot - 1, kt + S - 1);
                slice(kt, T_(), std::integral_constant<int, (S - 2) * L>());
            }
            drain<S - 2>([&](auto r) {        // slices kt + 1 .. nk - 1 are in flight
                constexpr int R = decltype(r)::value;
                if (nk - 1 - kt >= R) {
                    slice(kt, T_(), std::integral_constant<int, (R - 1) * L>());
                    ++kt;
                }
            });
        }
        // persistent: the block's next tile takes its first slice into slot 0 now -- every wave
        // finished reading slot 0 (slice nk - 2) before the last barrier -- so that it lands while
        // this tile's last slice and epilogue run
        const int nbid = bid + stride;
        static_assert(!PERSIST || S == 2, "the slot copied into ahead assumes a 2-stage ring");
        const bool more = PERSIST && nk % 2 == 0 && nbid < active;
        int ntm = 0, ntn = 0;
        if (more) {
            setup(nbid, ntm, ntn);
            issue(0, 0);
            issue_bias(ntn);
        }
        if constexpr (!AHEAD) slice(kt, F_(), std::integral_constant<int, 0>());   // last slice

        __syncthreads();   // every wave is done with the LDS ring
        // (persistent: the slabs sit past slot 0, which holds the next tile's first slice)
        float* const slabs = (float*)(PERSIST ? sm + STAGE : sm);
        epilogue_lds<E, TI, TJ>(a, acc, slabs + wave * (32 * (TJ * 32 + 4)),
                                m0 + tm * BM + wm * WM, tn * BN + wn * WN, M, lane);
        if (!more) {
            if (!PERSIST || nbid >= active) break;
            // an odd number of slices: nothing was copied ahead
            __builtin_amdgcn_s_waitcnt(0xc07f);
            bare_barrier();   // every wave is done with its slab
            bid = nbid;
            setup(bid, tm, tn);
            issue(0, 0);
            issue_bias(tn);
            wait_vm<0>();
            bare_barrier();
            continue;
        }
        bid = nbid;
        tm = ntm;
        tn = ntn;
        // the next tile's first slice and bias have landed -- every epilogue issues at least its
        // TI * NQ stores after their copies, and the stores need not be waited for -- and every
        // wave is done with its slab
        wait_vm<TI * (32 / (64 / (TJ * 8)))>();
        bare_barrier();
    }
}

// LDS of one block tile: the DMA ring, reused by the epilogue's per-wave slabs
template <int BM, int BN, int S, int WGM, int WGN>
constexpr size_t pipe_lds_bytes() {
    constexpr size_t ring = (size_t)S * (BM + BN) * 64 * 2;
    constexpr size_t slabs = (size_t)WGM * WGN * 32 * (BN / WGN + 4) * 4;
    return ring > slabs ? ring : slabs;
}
constexpr size_t PIPE_LDS = 160 * 1024;   // all of a compute unit's LDS: one workgroup per unit

// The tiles BM x BN of the rows [m0, M), walked by the grid one at a time.
template <Epi E, int BM, int BN, int S, int WGM, int WGN, bool AHEAD>
__device__ __forceinline__ void walk_tiles(const GemmArgs& a, uint16_t* sm, int m0, int M, int wave) {
    static_assert(pipe_lds_bytes<BM, BN, S, WGM, WGN>() <= PIPE_LDS, "LDS");
    if (wave >= WGM * WGN) return;
    const int n = (M - m0 + BM - 1) / BM * (a.Nout / BN);
    for (int t = blockIdx.x; t < n; t += gridDim.x) {
        pipe_tile<E, BM, BN, 64, S, WGM, WGN, false, AHEAD>(a, sm, t, m0, M, wave);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        bare_barrier();   // every wave is done with its slab: the next tile's copies may land
    }
}

// One workgroup per compute unit (the grid), tiles blockIdx.x, blockIdx.x + gridDim.x, ... of the
// large tiles over the rows [0, head), then of the plan's smaller tiles over [head, M).  BN: width
// of the large tiles.  The ring depths fill LDS: a small tile is bound by the latency of its loads.
// Measured against one workgroup per tile, the last round in 64 x 64 tiles up to a quarter of it
// and 128 x 128 up to half (us, before -> after; widths 1024, K = 4096 for FC2): FC2 at 340 / 700 /
// 2056 rows 26.1 -> 16.3, 27.0 -> 16.9, 54.2 -> 31.4; QKV at 700 rows 18.6 -> 11.0; out-projection at
// 2056 19.2 -> 12.6; at 37120 rows FC2 341 -> 311, out-projection 132 -> 124, FC1 305 -> 291.
// Large launches: QKV-shaped products of K = 4096 run 1288 TFLOP/s on random operands (hipBLASLt 1309) and
// 1484 on zeros (1943).  On random operands, where switching power lowers the clock, the kernel is
// within 2 % of the library; on zeros its own schedule holds it, so power is not its only limit.
template <Epi E, int BN>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_bf16_pipe_k(GemmArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    uint16_t* sm = (uint16_t*)smem;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: scalar LDS addresses
    const int M = a.Mdev ? *a.Mdev : a.Mconst;
    const GemmPlan p = gemm_plan(M, a.Nout, BN, gridDim.x, a.div_grid, a.div_tn, out_bytes(E));
    if (p.head > 0) {
        if constexpr (BN == 256) {
            pipe_tile<E, 256, 256, 64, 2, 2, 4, true>(a, sm, blockIdx.x, 0, p.head, wave, gridDim.x);
            __builtin_amdgcn_s_waitcnt(0xc07f);
            bare_barrier();
        } else {
            walk_tiles<E, 256, 128, 3, 4, 2, false>(a, sm, 0, p.head, wave);
        }
    }
    switch (p.tail) {
        case TAIL_192x256:
            if constexpr (BN == 256) walk_tiles<E, 192, 256, 2, 2, 4, false>(a, sm, p.head, M, wave);
            break;
        case TAIL_128x256:
            if constexpr (BN == 256) walk_tiles<E, 128, 256, 3, 2, 4, false>(a, sm, p.head, M, wave);
            break;
        case TAIL_128x128: walk_tiles<E, 128, 128, 5, 2, 4, false>(a, sm, p.head, M, wave); break;
        case TAIL_64x128: walk_tiles<E, 64, 128, 6, 2, 4, true>(a, sm, p.head, M, wave); break;
        case TAIL_64x64: walk_tiles<E, 64, 64, 9, 2, 2, true>(a, sm, p.head, M, wave); break;
        default: break;
    }
}

template <Epi E, int BN>
void launch_pipe(const GemmArgs& a0, hipStream_t s) {
    auto k = gemm_bf16_pipe_k<E, BN>;
    [[maybe_unused]] static const bool allowed = allow_lds((const void*)k, PIPE_LDS);
    // one block per compute unit, or per smallest tile when there are fewer
    const int tiles = ((a0.Mmax + 63) / 64) * (a0.Nout / 64);
    const int grid = std::min(tiles, a0.cus > 0 ? a0.cus : 256);
    if (grid <= 0) return;
    GemmArgs a = a0;
    a.div_grid = div_magic(grid);
    a.div_tn = div_magic(a.Nout / BN);
    hipLaunchKernelGGL(k, dim3(grid), dim3(512), PIPE_LDS, s, a);
}

// ---------------- fp32 MFMA GEMM ---------------------------------------------------------------
// v_mfma_f32_16x16x4_f32 (fp32 products and sums).  A block of four wavefronts (2 x 2) takes tiles of
// 32W x 32W, each wavefront W x W tiles of 16 x 16; k-slices of 32 floats go through the same kind of
// LDS ring as the bf16 path's (128-byte rows, the same swizzle).  Lane l reads 16 bytes of row l%16:
// k = 16 ks + 4 (l/16) + t for t = 0..3, its operands of four MFMAs, on both sides alike.  The weights
// are the first operand, so lane l ends with four consecutive columns of token row l%16.  Every
// output is four chains of MFMAs (one per t) in k order, added at the end, whatever the tile.
// Bound by the fp32 matrix rate (256 FLOP per clock and compute unit; 64 x 64 tiles need 16 bytes of
// operands per clock), or, in small models, by latency: 32 x 32 tiles spread few rows over more units.
// Against 64 x 64 tiles of VALU products (us): FC2 of width 768, about 1200 rows 299 -> 49, FC1 122 ->
// 41, QKV 127 -> 32; FC2 of width 192, 300 rows 78 -> 9.8.  Distance to 64-bit results halved.
constexpr size_t F32_LDS = 64 * 1024;   // two blocks per compute unit

template <Epi E, int W, int S>
__device__ __forceinline__ void f32_tile(const GemmArgs& a, float* sm, int t, int M, int wave) {
    constexpr int BT = 32 * W, BK = 32, RPI = 8, LR = BT / RPI / 4, L = 2 * LR;
    constexpr int STAGE = 2 * BT * BK;
    static_assert((size_t)S * STAGE * 4 <= F32_LDS, "LDS");
    int tm, tn;
    tile_coords(t, (M + BT - 1) / BT, a.Nout / BT, tm, tn);
    const int lane = threadIdx.x & 63, lr = lane & 15, g = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    const int K = a.K, nk = K / BK;
    uint32_t goffA[LR], goffB[LR];
#pragma unroll
    for (int u = 0; u < LR; ++u) {
        const int r = (wave * LR + u) * RPI + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        const int grow = tm * BT + r;
        const int arow = a.a_idx ? (grow < M ? a.a_idx[grow] : 0) : grow;   // gathered A rows
        goffA[u] = ((uint32_t)arow * K + c * 4) * 4;
        goffB[u] = ((uint32_t)r * K + c * 4) * 4;
    }
    const auto rA = buf_rsrc(a.A, BUF_ANY);
    const auto rW = buf_rsrc((const char*)a.W + (uint64_t)(uint32_t)(tn * BT) * (uint32_t)(K * 4), BUF_ANY);
    f32x4 acc[4][W][W];   // a chain per t: independent MFMAs, and shorter sums to round
    f32x4 bias[W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
        bias[j] = *(const f32x4*)(a.bias + tn * BT + (wn * W + j) * 16 + g * 4);
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    auto issue = [&](int kt) {
        float* st = sm + (kt % S) * STAGE;
#pragma unroll
        for (int u = 0; u < LR; ++u) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rW,
                (__attribute__((address_space(3))) void*)(st + (BT + (wave * LR + u) * RPI) * BK), 16,
                (int)goffB[u], kt * BK * 4, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rA,
                (__attribute__((address_space(3))) void*)(st + (wave * LR + u) * RPI * BK), 16,
                (int)goffA[u], kt * BK * 4, 0, 0);
        }
    };
    auto multiply = [&](int kt) {
        const float* st = sm + (kt % S) * STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            f32x4 xa[W], xb[W];
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const int ra = (wm * W + i) * 16 + lr, rb = (wn * W + i) * 16 + lr, c = ks * 4 + g;
                xb[i] = *(const f32x4*)(st + (BT + rb) * BK + (c ^ ((rb >> 1) & 7)) * 4);
                xa[i] = *(const f32x4*)(st + ra * BK + (c ^ ((ra >> 1) & 7)) * 4);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < W; ++i)
#pragma unroll
                    for (int j = 0; j < W; ++j)
                        acc[e][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(xb[j][e], xa[i][e],
                                                                            acc[e][i][j], 0, 0, 0);
        }
    };
#pragma unroll
    for (int p = 0; p < S - 1; ++p)
        if (p < nk) issue(p);
    int kt = 0;
    for (; kt + S - 1 < nk; ++kt) {
        wait_vm<(S - 2) * L>();   // slice kt has landed; this wave's reads of slice kt - 1 are done
        bare_barrier();
        issue(kt + S - 1);        // into the slot of slice kt - 1
        multiply(kt);
    }
    drain<S - 1>([&](auto r) {    // slices kt .. nk - 1 are in flight
        constexpr int R = decltype(r)::value;
        if (nk - kt >= R) {
            wait_vm<(R - 1) * L>();
            bare_barrier();
            multiply(kt);
            ++kt;
        }
    });
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int row = tm * BT + (wm * W + i) * 16 + lr;
        if (row >= M) continue;
#pragma unroll
        for (int j = 0; j < W; ++j)
            epi_store4<E>(a, row, tn * BT + (wn * W + j) * 16 + g * 4,
                          (acc[0][i][j] + acc[1][i][j]) + (acc[2][i][j] + acc[3][i][j]) + bias[j]);
    }
}

template <Epi E>
__global__ __launch_bounds__(256) void gemm_f32_k(GemmArgs a) {
    __shared__ __attribute__((aligned(16))) float sm[F32_LDS / 4];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int M = a.Mdev ? *a.Mdev : a.Mconst;
    // 32 x 32 tiles unless as many 64 x 64 tiles as the compute units take in as short a time: a
    // quarter of the work each, about a tenth more for operand traffic and barriers
    const int t64 = (M + 63) / 64 * (a.Nout / 64), t32 = (M + 31) / 32 * (a.Nout / 32);
    const int r64 = div_by(t64 + a.cus - 1, a.div_grid), r32 = div_by(t32 + a.cus - 1, a.div_grid);
    const bool large = r64 * 40 <= r32 * 11;
    const int n = large ? t64 : t32;
    for (int t = blockIdx.x; t < n; t += gridDim.x) {
        if (large) f32_tile<E, 2, 4>(a, sm, t, M, wave);
        else f32_tile<E, 1, 8>(a, sm, t, M, wave);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        bare_barrier();   // every wave has read its last slice: the next tile's copies may land
    }
}

template <Epi E>
void launch_one(bool bf16, const GemmArgs& a, hipStream_t s) {
    if (!bf16) {
        GemmArgs f = a;
        if (f.cus <= 0) f.cus = 256;
        f.div_grid = div_magic(f.cus);
        const int grid = std::min(((a.Mmax + 31) / 32) * (a.Nout / 32), 2 * f.cus);
        if (grid > 0) hipLaunchKernelGGL(gemm_f32_k<E>, dim3(grid), dim3(256), 0, s, f);
        return;
    }
    if (a.Nout % 256 == 0) launch_pipe<E, 256>(a, s);
    else launch_pipe<E, 128>(a, s);
}

}  // namespace

void launch_gemm(Epi e, bool bf16, const GemmArgs& a, hipStream_t s) {
    switch (e) {
        case Epi::Patch: launch_one<Epi::Patch>(bf16, a, s); break;
        case Epi::Qkv: launch_one<Epi::Qkv>(bf16, a, s); break;
        case Epi::OProj: launch_one<Epi::OProj>(bf16, a, s); break;
        case Epi::Fc1: launch_one<Epi::Fc1>(bf16, a, s); break;
        case Epi::Fc2: launch_one<Epi::Fc2>(bf16, a, s); break;
        case Epi::Restore: launch_one<Epi::Restore>(bf16, a, s); break;
        case Epi::Delta: launch_one<Epi::Delta>(bf16, a, s); break;
    }
}

}  // namespace dv
