// The launch rules of the kernels (host code of their headers) under C names, for test_plans.py.
#include <map>
#include <vector>

#include "attn_plan.h"

using namespace dv;

static int cut(int M, int Nout, int esz, int cus, int* head) {
    const int hbn = Nout % 256 == 0 ? 256 : 128;
    const int tiles = (M + 63) / 64 * (Nout / 64), slots = tiles < cus ? tiles : cus;
    const GemmPlan p = gemm_plan(M, Nout, hbn, slots, div_magic(slots), div_magic(Nout / hbn), esz);
    *head = p.head;
    return p.tail;
}

extern "C" {

// tail shape of the bf16 GEMM's plan; *head: rows in large tiles
int t_gemm_plan(int M, int Nout, int cus, int* head) { return cut(M, Nout, 4, cus, head); }

// the tail rows of a plan whose 32-bit offset in a packed output falls on a live row
long long t_stray_rows(int M, int Nout, int esz, int cus) {
    int head;
    const int tail = cut(M, Nout, esz, cus, &head);
    const int bm[] = {256, 192, 128, 128, 64, 64};
    const int from = tail == TAIL_NONE ? 0 : head, h = bm[tail];
    const int end = from + (M - from + h - 1) / h * h;
    long long n = 0;
    for (int r = M; r < end; ++r)
        for (uint32_t col : {0u, (uint32_t)Nout - 4})
            n += ((uint32_t)r * Nout + col) * esz < (unsigned long long)M * Nout * esz;
    return n;
}

// route of a bf16 attention launch; out: blocks, bytes of LDS, rows of other frames
int t_attn_plan(int dh, int F, int N, int H, int G, int star, int cus, long long* out) {
    AttnArgs a{};
    a.F = F;
    a.N = N;
    a.D = H * dh;
    a.H = H;
    a.G = G;
    a.star = star != 0;
    a.cus = cus;
    const AttnPlan p = dh == 64 ? attn_plan<64>(a) : dh == 80 ? attn_plan<80>(a)
                     : dh == 96 ? attn_plan<96>(a) : attn_plan<128>(a);
    out[0] = p.grid;
    out[1] = (long long)p.lds;
    out[2] = p.pcap;
    return p.route;
}

// grid of the streamed kernel, or -1 unless its blocks take every (frame from skip on, head, block of
// the frame) exactly once and nothing else; *together: blocks that share an XCD with their unit's first
long long t_stream_grid(int F, int skip, int N, int H, int G, long long* together) {
    const StreamMap m(F, skip, N, H, G);
    std::vector<int> seen((size_t)F * H * m.qblocks, 0);
    std::map<int, int> xcd;
    *together = 0;
    for (int b = 0; b < m.grid; ++b) {
        int f, h, qb;
        if (!m.item(b, f, h, qb)) continue;
        if (f < skip || f >= F || h < 0 || h >= H || qb < 0 || qb >= m.qblocks) return -1;
        if (seen[((size_t)f * H + h) * m.qblocks + qb]++) return -1;
        const int unit = f / (G > 0 ? G : 1) * H + h;
        *together += xcd.emplace(unit, b % 8).first->second == b % 8;
    }
    long long n = 0;
    for (int s : seen) n += s;
    return n == (long long)(F - skip) * H * m.qblocks ? m.grid : -1;
}
}
