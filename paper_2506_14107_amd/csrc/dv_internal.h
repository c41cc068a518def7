// Internal interface between the orchestrator (api.hip) and the kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace dv {

// Lets kernel `k` be launched with `bytes` of dynamic LDS.  Called to initialise a static local of its
// launcher: once, also when several host threads launch for the first time together.
inline bool allow_lds(const void* k, size_t bytes) {
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess;
}

// ---- bf16 storage helpers (raw 16-bit patterns) ---------------------------------------------
__host__ __device__ inline uint16_t f32_to_bf16(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest, ties to even (finite inputs)
    return (uint16_t)(u >> 16);
}
__host__ __device__ inline float bf16_to_f32(uint16_t h) {
    return __builtin_bit_cast(float, (uint32_t)h << 16);
}

// ---- reordered referencing (I/P/B frames with past and future references) --------------------
// Groups of G frames (G a multiple of 4) start with an I frame, computed in full.  Positions
// 4, 8, ... of a group are P frames referencing the anchor four frames back.  Between two
// anchors a and a + 4 (the next group's I frame closes the group's last block) the frame at
// a + 2 is B_dist2, referencing both anchors, and those at a + 1 and a + 3 are B_dist1,
// referencing their neighbours among a, a + 2, a + 4.  A reference at or past frame F (the
// end of the frames at hand) is absent (-1).  type: 0 I, 1 P, 2 B_dist2, 3 B_dist1.
struct FrameRefs {
    int type, past, fut;
};
__host__ __device__ inline FrameRefs reorder_refs(int f, int G, int F) {
    const int p = f % G;
    if (p == 0) return {0, -1, -1};
    const int d = p & 3, a = f - d;
    FrameRefs q;
    if (d == 0) q = {1, f - 4, -1};
    else if (d == 2) q = {2, a, a + 4};
    else if (d == 1) q = {3, a, a + 2};
    else q = {3, a + 2, a + 4};
    if (q.fut >= F) q.fut = -1;
    return q;
}

// ---- GEMM ------------------------------------------------------------------------------------
// C[M, Nout] = A[M, K] * W[Nout, K]^T with a fused epilogue.  M is read on the device.
enum class Epi : int {
    Patch = 0,  // x[(r/P)*N + 1 + r%P, c] = acc + bias[c] + pos[(1 + r%P), c]        (fp32 out)
    Qkv = 1,    // qkv[r, c] = acc + bias[c]                                           (elem out)
    OProj = 2,  // z[r, c] = acc + bias[c] + x[idx[r], c]                              (fp32 out)
    Fc1 = 3,    // h[r, c] = gelu(acc + bias[c])                                       (elem out)
    Fc2 = 4,    // x[idx[r], c] = acc + bias[c] + z[r, c]                              (fp32 out)
    Restore = 5,  // x[t, c] = acc + bias[c] + x[ref(t), c], t = idx[r]: a reused token's row
                  // from its reference token's new row (ref(t): same token of frame G*floor(f/G))
    Delta = 6,    // out[r, c] = acc + bias[c]                                        (fp32 out)
};

struct GemmArgs {
    const void* A;       // [rows, K] row-major; rows padded to the tile height
    const void* W;       // [Nout, K] row-major
    const float* bias;   // [Nout]
    int K, Nout;
    const int* Mdev;     // device row count (nullptr: use Mconst)
    int Mconst;
    int Mmax;            // upper bound on M (grid sizing)
    void* out;
    const float* resid;  // OProj: x rows; Fc2: z rows
    const int* idx;      // packed row -> token row
    const int* a_idx;    // A row gather: packed row m reads A row a_idx[m] (nullptr: row m)
    const float* pos;    // Patch: position table [N, D]
    int P, N;            // Patch: patches and tokens per frame (Restore: N)
    int G;               // Restore: group size
    int cus;             // compute units of the device (0: unknown)
    // set by the launcher: division by the grid (fp32: by the compute units) and by the large tile
    // columns
    uint32_t div_grid, div_tn;
};

// n / d for n < 2^24, d < 2^8 or so (n * d < 2^32) by one multiplication with div_magic(d): a
// kernel's few divisions by values known at launch, which the hardware would do in dozens of
// instructions each.  div_magic(1) = 0 stands for 2^32.
inline uint32_t div_magic(uint32_t d) { return d == 1 ? 0u : (uint32_t)((0x100000000ull + d - 1) / d); }
__host__ __device__ inline int div_by(int n, uint32_t magic) {
    return magic ? (int)(((uint64_t)(uint32_t)n * magic) >> 32) : n;
}

// Records of a buffer descriptor whose offsets are all valid, and an offset that no buffer holds.
constexpr uint32_t BUF_ANY = 0xFFFFFFF0u;

// How the M rows of a bf16 GEMM are cut: large tiles (256 x hbn) over the rows [0, head) -- the
// tile rows that fill whole rounds of `slots` workgroups -- and one smaller tile shape over
// [head, M), the rows of the last, partial round.  Each output is the same dot product in the same
// k order in any tile, so the plan does not change results.
// The partial round takes the shape with the least rounds x time per tile.  Times per tile,
// relative to a 256 x 256 tile, measured at K = 1024 and 4096 alike (per-launch overhead taken off,
// one tile per compute unit: FC2 of width 1024, us: 70 / 57 / 41 / 28 / 19 / 16.5 for 256 x 256,
// 192 x 256, 128 x 256, 128 x 128, 64 x 128, 64 x 64; the last is 13 since its copies follow its
// reads, which changes no choice between whole rounds): the smaller the tile, the more of it is the
// latency of its loads, barriers and epilogue.
enum GemmTail : int {
    TAIL_NONE = 0, TAIL_192x256, TAIL_128x256, TAIL_128x128, TAIL_64x128, TAIL_64x64
};
struct GemmPlan {
    int head;
    int tail;
};
// 192-row tiles can end past the padding of the rows to 256, which bounds 32-bit offsets, by up to 128
// rows: they are left out where such a row's place in a packed output of `esz`-byte elements would pass 2^32
// and come out as that of a live row.  (That test, per tile row and store instead: ViT-B/16, 64 frames,
// 0.5 % slower.)
__host__ __device__ inline GemmPlan gemm_plan(int M, int Nout, int hbn, int slots, uint32_t div_slots,
                                              uint32_t div_tn, uint32_t esz) {
    const int tn = Nout / hbn;
    const int mt = (M + 255) / 256;
    const int mA = div_by(div_by(mt * tn, div_slots) * slots, div_tn);   // whole tile rows inside the full rounds
    GemmPlan p = {M, TAIL_NONE};
    if (mA >= mt) return p;
    const int rows = M - mA * 256;
    int best = hbn == 256 ? 100 : 59;                // the partial round in large tiles
    auto consider = [&](int kind, int bm, int bn, int cost) {
        const int tiles = (rows + bm - 1) / bm * (Nout / bn);
        const int c = div_by(tiles + slots - 1, div_slots) * cost;
        if (c < best) {
            best = c;
            p.head = mA * 256;
            p.tail = kind;
        }
    };
    if (hbn == 256) {
        const uint32_t past = (uint32_t)(M + 191);   // the last row of a 192-row tile, at most
        if ((uint64_t)past * ((uint32_t)Nout * esz) < BUF_ANY) consider(TAIL_192x256, 192, 256, 81);
        consider(TAIL_128x256, 128, 256, 59);
    }
    consider(TAIL_128x128, 128, 128, 39);
    consider(TAIL_64x128, 64, 128, 27);
    consider(TAIL_64x64, 64, 64, 23);
    return p;
}

void launch_gemm(Epi e, bool bf16, const GemmArgs& a, hipStream_t s);
// Measurement probe: `blocks` blocks of 256 threads run `iters` rounds of four independent bf16
// MFMA chains; returns the FLOPs the launch performs.  sink: blocks*256 floats.
double launch_mfma_loop(int blocks, int iters, float* sink, hipStream_t s);

// ---- attention -------------------------------------------------------------------------------
struct AttnArgs {
    const void* qkv;   // packed rows [M, 3D] (Q | K | V), elem
    const int* pos;    // [F*N] packed row of each token's K/V (reused -> reference's row)
    const int* qoff;   // [F+1] packed query rows of frame f: qoff[f] .. qoff[f+1]
    void* out;         // [M, D] elem
    int F, N, D, H;
    int G;             // group size, 0 without reuse
    int cus;           // compute units of the device (0: unknown)
    int skip;          // leading frames carried over from an earlier call (no rows, no queries)
    bool star;         // every frame's reused keys are its group's first frame's, packed in this batch
};
void launch_attention(bool bf16, const AttnArgs& a, hipStream_t s);
// Class-token attention weights of every non-reference frame (G > 0: frames f % G == 0 are
// skipped), per head: probs[(f*H + h)*N + j] = softmax_j(q_h . k_h,j / sqrt(dh)) with q the
// frame's class-token query (its first packed row, qoff[f]) and k_j its key row through pos.
void launch_cls_attention(bool bf16, const AttnArgs& a, float* probs, hipStream_t s);
size_t attention_lds_bytes(bool bf16, int N, int dh);
bool attention_supported(bool bf16, int N, int dh);

// ---- row kernels -----------------------------------------------------------------------------
// Patch rows A of F frames, and their class-token rows x[f, 0, :] = cls + pos[0] (N = P + 1 rows of D
// per frame)
void launch_im2col(bool bf16, const float* frames, int F, int S, int p, int Kp, void* A, float* x,
                   const float* cls, const float* pos, int D, int cus, hipStream_t s);

// Weight matrices that launches soon after read, touched once by wavefronts of a row kernel that have
// nothing else to do (every 128-byte line once, 4 bytes of it), so that small GEMMs, bound by the
// latency of their loads, find them on the die instead of in HBM.  n = 0: nothing to touch.
struct Touch {
    const void* p[2];
    uint32_t lines[2];   // 128-byte lines
    int n;
};

enum GateMode : int { GATE_COS = 0, GATE_INJECT = 1, GATE_ALL = 2, GATE_NONE = 3 };
struct GateArgs {
    float* x;             // [F*N, D] (written only to give a recomputed alias its row)
    int F, N, D, G, L, layer;
    int mode;
    float tau;
    const uint8_t* prev;  // previous layer's map (gate mode, monotone shortcut) or nullptr
    const uint8_t* inj;   // injected maps [F, L, N] (batch base) or nullptr
    uint8_t* cur;         // [F*N] this layer's map (or nullptr)
    uint8_t* out_masks;   // [F, L, N] (batch base) or nullptr
    int* cnt;             // [F * gate_chunks(N)] recomputed tokens per block (or nullptr)
    const float* ln_g;    // LN1 gain / shift
    const float* ln_b;
    void* ln_out;         // [F*N, D] elem: LN1 rows of recomputed tokens (token-indexed) or nullptr
    void* d_out;          // [F*N, D] elem: x_f - x_ref rows of reused tokens (token-indexed;
                          // restoration) or nullptr.  May be ln_out: the rows are disjoint.
    const float* dec;     // GATE_COS with the decision MLP: the layer's W_d1 [64,6], b_d1 [64],
                          // W_d2 [64], b_d2 [1] (fp32, back to back), else nullptr
    const float* tcls;    // [F, H, N] class-token attention weights of the previous layer, per
                          // head (nullptr: 1/N); the cue is their mean over the H heads
    int H;
    int reorder;          // reordered referencing (reorder_refs) instead of the star
    uint8_t* src;         // [F*N] reordered: 1 where the future reference supplies the token
    const int* root;      // [F*N] reordered: the previous layer's root map (nullptr: every token
                          // holds its own row); a recomputed token gets its root's row copied in
    int skip;             // leading frames carried over from an earlier call of a stream: one is
                          // the cached reference (the first in the star, the last under
                          // reordering; its rows already in x), the others gaps; none is gated,
                          // and inj / out_masks start at frame skip
    int cus;              // compute units of the device (0: unknown)
    Touch touch;          // small batches only (a wavefront per token)
};
// Reordering with restoration: a reused row is built along its chain of sources; a group of G
// frames has chains of at most G/4 + 1 reused links (B_dist1, B_dist2, then the P frames back
// to the I frame), so G <= 4 * (CHAIN_MAX - 1).
constexpr int CHAIN_MAX = 16;
constexpr int DEC_HIDDEN = 64;   // decision MLP hidden units: one per lane of a wavefront
constexpr int DEC_FEAT = 6;      // its features: s, t, one-hot type (I, P, B_dist2, B_dist1)
constexpr int DEC_FLOATS = DEC_HIDDEN * DEC_FEAT + 2 * DEC_HIDDEN + 1;
// Mode GATE_NONE marks every token recomputed (reuse off) and only writes LN1 rows.
// The gate runs in blocks of GATE_TOK tokens; counts are per block: cnt[f * gate_chunks(N) + c].
constexpr int GATE_TOK = 16;
inline int gate_chunks(int N) { return (N + GATE_TOK - 1) / GATE_TOK; }
void launch_gate(bool bf16, const GateArgs& a, hipStream_t s);
void launch_count(const uint8_t* m, int F, int N, int G, int* cnt, hipStream_t s);
// qoff[0..F] = exclusive prefix of the per-frame counts (sum of `per` consecutive entries of
// cnt per frame), M[0] = qoff[F]; M[1] = tokens - M[0] (the reused tokens) when tokens > 0
void launch_scan(const int* cnt, int per, int F, int tokens, int* qoff, int* M, hipStream_t s);
// idx/pos from a per-layer map and its qoff (cur == nullptr: every token recomputed, identity
// lists, qoff_in ignored and qoff_out written)
// ridx (or nullptr): the reused tokens f*N+i of non-reference frames in frame-major order, at
// slot (f*N - qoff[f]) + (reused tokens of frame f before i)
// skip > 0 (stream): frames below skip have no rows; one of them is the cached reference (the
// first in the star, the last under reordering), whose keys and values sit at packed rows
// ext_row .. ext_row + N - 1: pos of every token of those frames points there
// rslot (or nullptr): for every reused token, its slot in ridx
void launch_compact(const uint8_t* cur, const int* qoff_in, int F, int N, int G, int* idx,
                    int* pos, int* qoff_out, int* ridx, hipStream_t s, int skip = 0,
                    int ext_row = 0, int* rslot = nullptr);
// launch_scan then launch_compact in one launch: every block sums the per-block counts of the
// frames before it (and before its reference) itself; qoff, M as launch_scan writes them
void launch_scan_compact(const int* cnt, int per, int tokens, const uint8_t* cur, int F, int N,
                         int G, int* idx, int* pos, int* qoff, int* M, int* ridx, hipStream_t s,
                         int skip = 0, int ext_row = 0, int* rslot = nullptr);
// dst[i, 0:2D] = K|V of packed row pos[f*N + i], el-byte elems
void launch_copy_ref_kv(const void* qkv, const int* pos, int f, int N, int D, int el, void* dst,
                        hipStream_t s);
// dst[i, 0:D] = x row of token i of frame root[f*N + i] (root == nullptr: of frame f)
void launch_copy_rows(const float* x, const int* root, int f, int N, int D, float* dst,
                      hipStream_t s);

// LayerNorm of rows (optionally gathered through idx) into elem rows: dst[r] = LN(src[g(r)])
void launch_ln_rows(bool bf16, const float* src, const int* gather, const int* Mdev, int Mmax,
                    int D, const float* g, const float* b, void* dst, const Touch& touch,
                    hipStream_t s);
// x[f*N+i] = x[r*N+i] for every token with cur[f*N+i] != 0, r = root[f*N+i] (root == nullptr:
// the group's first frame)
void launch_merge(float* x, const uint8_t* cur, const int* root, int F, int N, int D, int G,
                  hipStream_t s);
// Reordered referencing with the restoration layer: every reused token's new row, built along its
// chain of sources from the root's new row: x[t] = ((x[root] + d[link_1]) + ...) + d[t], where
// d[u] = rbuf[rslot[u]] is token u's restoration output and the links run from the root outward.
// Mdev: the number of reused tokens (rows of ridx).
void launch_restore_chain(float* x, const float* rbuf, const int* ridx, const int* rslot,
                          const uint8_t* cur, const uint8_t* src, const int* Mdev, int Mmax, int F,
                          int N, int D, int G, hipStream_t s);
// Reordered referencing: for every reused token, follow the sources (src, reorder_refs) to the
// frame r that recomputes it; pos[f*N+i] = pos[r*N+i], root[f*N+i] = r (f for recomputed ones).
void launch_resolve(const uint8_t* cur, const uint8_t* src, int F, int N, int G, int* pos,
                    int* root, hipStream_t s);
// emb[f] = LN(x[f*N]) (class token)
void launch_final_ln(const float* x, int F, int N, int D, const float* g, const float* b,
                     float* emb, hipStream_t s);

}  // namespace dv
