// Which bf16 attention kernel takes a launch, with which grid and how much LDS: functions of this launch's
// sizes alone, so that a launch costs the same whatever ran before it in the process.
#pragma once
#include <algorithm>

#include "dv_internal.h"

namespace dv {

constexpr size_t ATTN_LDS = 160 * 1024;   // LDS of a compute unit

// ---- LDS geometry of the bf16 kernels (shared by host sizing and the kernels) ------------------
// K rows: the MFMA reads 16 bytes (one chunk) of 16 consecutive rows; V rows: the transposing
// read ds_read_b64_tr_b16 reads 8 bytes (4 dims) of 4 consecutive keys x 4 dim-words.  Row
// strides and XOR swizzles (in 16-byte chunks) keep both patterns on distinct banks:
//   head dim 64:  K chunk c of row r at c ^ ((r>>1)&7),  V chunk c of row j at c ^ 2((j>>1)&3)
//   head dim 128: K chunk c of row r at c ^ (r&15),      V chunk c of row j at c ^ 2(j&3)
//   head dim 80/96: no swizzle; K rows padded to dh+8, V rows to 96 elements.
struct Geo {
    int npad, ldk, ldv, dh;
    __host__ __device__ Geo(int N, int d) : dh(d) {
        npad = (N + 31) / 32 * 32;
        ldk = (d == 64 || d == 128) ? d : d + 8;
        ldv = (d == 64 || d == 128) ? d : 96;
    }
    __host__ __device__ int kofs(int r, int c) const {
        const int x = dh == 64 ? ((r >> 1) & 7) : dh == 128 ? (r & 15) : 0;
        return r * ldk + (c ^ x) * 8;
    }
    __host__ __device__ int vofs(int j, int c) const {
        const int x = dh == 64 ? 2 * ((j >> 1) & 3) : dh == 128 ? 2 * (j & 3) : 0;
        return j * ldv + (c ^ x) * 8;
    }
    __host__ __device__ size_t bytes() const {
        return ((size_t)npad * ldk + (size_t)npad * ldv) * 2;
    }
};

// ---- blocks of the streamed kernel -------------------------------------------------------------
// A unit (a group's frames, one head) lives on one XCD, so that the XCD's L2 serves the reference rows
// its frames share: workgroups are dealt to the 8 XCDs round-robin.  The frames below `skip` have no
// queries and get no blocks, and neither do the places of a group that the batch does not fill: an
// empty block still waits for its LDS (4-frame calls of a ViT-L/14 stream in groups of 256, 24 layers,
// with blocks for whole groups: the first 1974 us, now 1872; the 64th 2586, now 2312).  Where whole
// units would leave more blocks empty than busy (few heads, a last group of a frame or two) every
// frame is a unit of its own.
// Many blocks: a unit's one after another.  Few (all resident at once): an XCD deals its blocks round its
// 32 compute units, so those that surely have queries -- the reference frames' -- come first, then
// the other frames' first blocks, then the rest, most of them empty under reuse: two busy ones meet on
// a unit only when more than 32 are busy.  One unit after another / this order, us a layer at 90 % reuse:
// ViT-L/14, 8 and 12 frames 10.1 / 7.9 and 9.4 / 8.3, at 336 px 4 frames 17.8 / 13.6; 26 heads, 3
// frames 10.2 / 8.3 (blocks for whole groups 9.9, 10.0, 16.9 and 8.3); 16 frames, 768 blocks, 10.3 / 10.5.
constexpr int FW = 4;   // wavefronts (query tiles) of a streamed block
struct StreamMap {
    int F, H, G, skip;
    int g0;        // the first unit's group
    int span;      // frames per unit, at most
    int qblocks;   // blocks per frame and head
    int per_xcd;   // units of an XCD where all blocks are resident at once, else 0
    int lead;      // 1 where a unit's first frame is its reference, computed in full
    int grid;
    StreamMap(int F_, int skip_, int N, int H_, int G_) : F(F_), H(H_), G(G_ > 0 ? G_ : 1), skip(skip_) {
        qblocks = ((N + 31) / 32 + FW - 1) / FW;
        deal();
        const int busy = (F - skip) * H * qblocks;
        if (G > 1 && (grid < 0 || grid > 2 * busy)) {
            G = 1;
            deal();
        }
    }
    // frame, head and block of the frame of grid index b; false: nothing to do
    __host__ __device__ bool item(int b, int& f, int& h, int& qb) const {
        int e = b / 8, k, j = 0;   // the XCD's k-th unit, the unit's j-th frame
        if (per_xcd > 0) {
            k = e % per_xcd;
            const int r = e / per_xcd - lead * qblocks;
            if (r < 0) {
                qb = r + qblocks;
            } else {
                qb = r / (span - lead);
                j = lead + r - qb * (span - lead);
            }
        } else {
            const int per = span * qblocks;
            k = e / per;
            e -= k * per;
            j = e / qblocks;
            qb = e - j * qblocks;
        }
        const int u = k * 8 + b % 8, g = g0 + u / H;
        f = (g * G > skip ? g * G : skip) + j;
        h = u % H;
        return f < F && f < (g + 1) * G;
    }

private:
    static constexpr int RESIDENT = 3 * 256;   // blocks: three to a compute unit (registers)
    void deal() {
        g0 = skip / G;
        lead = skip % G == 0;
        span = std::min(G, F - skip);
        const long long units = (long long)((F + G - 1) / G - g0) * H;
        const long long n = (units + 7) / 8 * 8 * span * qblocks;
        grid = n < (1ll << 31) ? (int)n : -1;
        per_xcd = n <= RESIDENT ? (int)((units + 7) / 8) : 0;
    }
};

// LDS of a per-unit block: K and V arrays of npad reference rows (keys past N repeat key N-1) followed
// by up to pcap rows of other frames; then one 16-bit key -> row map of npad entries per frame of
// the group.
struct UnitGeo {
    Geo g;
    int pcap, G;
    __host__ __device__ UnitGeo(int N, int dh, int G_, int pcap_) : g(N, dh), pcap(pcap_), G(G_) {}
    __host__ __device__ int rows() const { return g.npad + pcap; }
    __host__ __device__ size_t vbase() const { return (size_t)rows() * g.ldk; }   // elements
    __host__ __device__ size_t mbase() const { return vbase() + (size_t)rows() * g.ldv; }
    __host__ __device__ size_t bytes() const { return (mbase() + (size_t)G * g.npad) * 2; }
};

// Rows of other frames that fit in `limit` bytes of LDS next to the reference rows and maps.
inline int unit_pcap(int N, int dh, int G, size_t limit) {
    const UnitGeo u(N, dh, G, 0);
    const size_t per = (size_t)(u.g.ldk + u.g.ldv) * 2;
    return u.bytes() >= limit ? 0 : (int)std::min<size_t>((limit - u.bytes()) / per, 32767);
}

// ---- the rule ----------------------------------------------------------------------------------
// Which kernel: the same bits from each (one arithmetic per query), so the rule is about time alone.
//   per unit   head dim 64, star groups whose reference rows leave LDS for another frame's, and
//              units (groups x heads, one block per compute unit) that fill their rounds to 9/10: the
//              reference's keys are staged once per group.
//   per frame  more frames x heads than blocks are resident, and either head dim 64 with two
//              blocks' keys per compute unit (up to 320 keys) without reuse or in groups of at most 4,
//              or head dim 128 (one block; 64 frames of 8 heads at 90 % 31 us a layer, streamed 34).
//   streamed   everything else: few frames, ungrouped reuse (reordering, stream calls), head dims 80
//              and 96 or long key rows (a frame's keys fill most of LDS, eight wavefronts a unit).
// Measured, us a layer, streamed / per frame / per unit (bf16, ViT-L/14 unless named): 256 frames
// in groups of 8 at 50 % reuse 143 / - / 127, 90 % 80 / 143 / 57; 192 frames (1.5 rounds of units) 113 /
// - / 138 and 73 / - / 68; 64 frames 42 / - / 64 and 29 / - / 33; reuse off, 8 frames 15 / 16 (66 without
// several blocks to a frame), 128 frames 121 / 105; 336 px (577 keys) 60 % 168 / 222 / -, 90 % 94 / 140;
// ViT-H/14 (head dim 80) 53 / 62; ViT-B/16, 64 frames in groups of 4, 24.5 / 22.5 / 25.7; reordered 256
// frames at 90 % 86 / 114 (with a streaming wavefront per tile for short frames).
enum AttnRoute : int { ATTN_STREAM = 0, ATTN_FRAME, ATTN_UNIT };
struct AttnPlan {
    int route;
    int grid;      // blocks (per frame, per unit)
    size_t lds;    // bytes of LDS a block
    int pcap;      // per unit: rows of other frames
};
// Blocks of the per-frame kernel that a compute unit holds: its registers allow 16 wavefronts at head
// dim 64 (two blocks of eight; the rule gives it launches whose keys fit LDS twice) and 8 at 128.  The
// other head dims have no per-frame kernel.
constexpr int frame_blocks(int dh) { return dh == 64 ? 2 : dh == 128 ? 1 : 0; }

template <int DH>
AttnPlan attn_plan(const AttnArgs& a) {
    const int items = a.F * a.H, resident = frame_blocks(DH) * a.cus;
    const size_t lds = Geo(a.N, DH).bytes();
    if (DH == 64 && a.star && a.G > 1 && a.cus > 0) {
        const int units = (a.F + a.G - 1) / a.G * a.H;
        const int pcap = unit_pcap(a.N, DH, a.G, ATTN_LDS);
        if (pcap >= a.N && units * 10 >= (units + a.cus - 1) / a.cus * a.cus * 9)
            return {ATTN_UNIT, std::min(units, a.cus), UnitGeo(a.N, DH, a.G, pcap).bytes(), pcap};
    }
    bool frame = resident > 0 && items > resident;
    if (DH == 64) frame = frame && 2 * lds <= ATTN_LDS && (a.G <= 1 || (a.star && a.G <= 4));
    if (frame) return {ATTN_FRAME, resident, lds, 0};
    const Geo g(a.N, DH);
    return {ATTN_STREAM, 0, (size_t)128 * (g.ldk + g.ldv) * 2, 0};
}

}  // namespace dv
