// Front-to-back compositing (Eq. 2) and its backward -- gfx950.
//
// Four wave64s per 16x16 tile, each owning an 8x8 quadrant (one pixel per
// lane) and walking the tile's depth-ordered list independently.  Records
// are staged in LDS in chunks of 64, culled against the quadrant with each
// record's alpha box and compacted by ballot; all lanes then read the same
// staged record, which the LDS serves as a broadcast.  The forward keeps no
// per-pixel lists: it stores the final transmittance and the position of the
// last composited entry, and the backward walks the list back to front,
// recovering T_i = T_{i+1} / (1 - alpha_i).
//
// Backward: the gradient fields of an entry are sums over a quadrant's pixels
// of products with two per-pixel values, which pass through LDS so that a lane
// sums a row of pixels of one entry in registers; after each chunk the wave
// adds the sums to the per-slot 2D gradient buffer with one float atomic per
// nonzero field.
#include "gs_internal.h"

namespace gs {

namespace {

// alpha of record (a, b) at pixel centre (px, py): the same instruction
// sequence in forward and backward, so skip and stop decisions agree bit
// for bit.
struct Eval {
    float dx, dy, G, raw, alpha;
    bool keep;   // not skipped (power <= 0 and alpha >= 1/255)
};

__device__ __forceinline__ Eval eval_entry(const float4 a, const float4 b, float px, float py) {
    Eval e;
    e.dx = px - a.x;
    e.dy = py - a.y;
    const float p2 = fmaf(a.z, e.dx * e.dx, fmaf(a.w, e.dx * e.dy, b.x * (e.dy * e.dy)));
    e.G = __builtin_amdgcn_exp2f(p2);
    e.raw = b.y * e.G;
    e.alpha = fminf(kAlphaMax, e.raw);
    e.keep = !(p2 > 0.0f) && e.alpha >= kAlphaMin;
    return e;
}

// Record -> LDS form: the mean relative to the tile origin (integer part
// minus the origin is exact; adding the stored fraction rounds once, at the
// scale of the tile rather than of the image).
__device__ __forceinline__ float4 stage_geom(const float4 r0, const float4 r1, const float4 r2, float ox, float oy) {
    return make_float4((r0.x - ox) + r1.w, (r0.y - oy) + r2.w, r0.z, r0.w);
}

// Four independent wave64s per 16x16 tile, one 8x8 quadrant each, one
// pixel per lane.  A wave walks the tile's list in chunks of 64: every lane
// gathers one record, tests the record's box (opacity' G' >= 1/255 region,
// with margins) against the wave's quadrant, and the ballot of survivors
// compacts them, in list order, into the wave's LDS slice.  The wave then
// evaluates only the survivors: an entry whose box misses every pixel of the
// quadrant has alpha < 1/255 there and would be skipped anyway, so results
// are unchanged while the horizon tiles' long lists of tiny, distant
// Gaussians cost a fraction of the work.  The per-entry update is predicated
// (selects, no branches).  Waves of a tile never wait for each other.
constexpr int kChunk = 64;
constexpr int kWaves = 4;

// the workgroup's tile: its place in the launch order (an order that is not
// a permutation of the tiles falls back to the index, so no access strays)
__device__ __forceinline__ int launch_tile(const uint32_t* __restrict__ tile_order, const ViewTable& vt) {
    const uint32_t t = tile_order ? tile_order[blockIdx.x] : blockIdx.x;
    return t < (uint32_t)vt.total_tiles ? (int)t : (int)blockIdx.x;
}

struct PixelCoords {
    int v;
    float ox, oy;          // tile origin in pixels
    float fpx, fpy;        // pixel centre relative to the tile origin
    float qcx, qcy;        // centre of the wave's quadrant (pixel-centre span +-3.5)
    bool inside;
    int64_t pix;
    int lx, ly;            // pixel within the tile
};

// a wave-uniform float in a scalar register (uniform float arithmetic is
// done by the vector unit and would hold a vector register for the whole walk)
__device__ __forceinline__ float uniform(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

__device__ __forceinline__ PixelCoords pixel_coords(const ViewTable& vt, int tile, int wave, int lane) {
    PixelCoords c;
    c.v = view_of_tile(vt, tile);
    const ViewK& V = vt.v[c.v];
    const int lt = tile - V.tile_off;
    const int ty = lt / V.tiles_x, tx = lt - ty * V.tiles_x;
    const int qx0 = (wave & 1) * 8, qy0 = (wave >> 1) * 8;
    const int lx = qx0 + (lane & 7), ly = qy0 + (lane >> 3);
    c.ox = uniform((float)(tx * kTile));
    c.oy = uniform((float)(ty * kTile));
    c.fpx = (float)lx + 0.5f;
    c.fpy = (float)ly + 0.5f;
    c.qcx = uniform((float)qx0 + 4.0f);
    c.qcy = uniform((float)qy0 + 4.0f);
    const int px = tx * kTile + lx, py = ty * kTile + ly;
    c.inside = px < V.W && py < V.H;
    c.pix = V.pix_off + (int64_t)py * V.W + px;
    c.lx = lx;
    c.ly = ly;
    return c;
}

// does the record's alpha box reach the wave's quadrant of pixel centres?
__device__ __forceinline__ bool box_hits_quadrant(const float4 g, const float4 r3, float qcx, float qcy) {
    const float mx = g.x, my = g.y;
    return fabsf(mx - qcx) <= r3.x + 3.5f + 1e-3f + 1e-6f * fabsf(mx) &&
           fabsf(my - qcy) <= r3.y + 3.5f + 1e-3f + 1e-6f * fabsf(my) && r3.x >= 0.0f;
}

// Does the entry's alpha reach 1/255 anywhere in the wave's quadrant?  The
// exponent p(d) = qa dx^2 + qb dx dy + qc dy^2 (d = pixel centre - mean) is a
// concave quadratic; its maximum over the rectangle spanned by the
// quadrant's pixel centres is 0 when the mean lies inside, otherwise the
// largest of the four edges' one-dimensional maxima.  The entry can only be
// composited where o' 2^p >= 1/255, i.e. p >= log2(1/(255 o')); the test is
// relaxed by 1e-5 and by 16 float32 ulps of the terms' magnitudes, which
// covers the rounding of both this test and the kernels' own evaluation of
// p, so an entry it rejects has alpha < 1/255 at every pixel of the quadrant.
// max over dy in [lo, hi] of qa dx^2 + qb dx dy + qc dy^2 (qc < 0), m = -qb /
// (2 qc): any dy gives a lower bound of the maximum, so the slope's rounding
// (one ulp of v_rcp_f32) costs |qc| (dy ulp)^2 at most, far inside the margin
__device__ __forceinline__ float edge_max(float qa, float qb, float qc, float m, float dx, float lo, float hi) {
    const float dy = fminf(fmaxf(m * dx, lo), hi);
    return fmaf(qa, dx * dx, fmaf(qb, dx * dy, qc * (dy * dy)));
}

__device__ __forceinline__ bool ellipse_hits_quadrant(const float4 g, const float4 r1, float qcx, float qcy) {
    const float qa = g.z, qb = g.w, qc = r1.x, o = r1.y;
    const float dx0 = (qcx - 3.5f) - g.x, dx1 = (qcx + 3.5f) - g.x;
    const float dy0 = (qcy - 3.5f) - g.y, dy1 = (qcy + 3.5f) - g.y;
    if (dx0 <= 0.0f && dx1 >= 0.0f && dy0 <= 0.0f && dy1 >= 0.0f) return true;
    const float hb = -0.5f * qb, my = hb * __builtin_amdgcn_rcpf(qc), mx = hb * __builtin_amdgcn_rcpf(qa);
    float m = fmaxf(edge_max(qa, qb, qc, my, dx0, dy0, dy1), edge_max(qa, qb, qc, my, dx1, dy0, dy1));
    m = fmaxf(m, fmaxf(edge_max(qc, qb, qa, mx, dy0, dx0, dx1), edge_max(qc, qb, qa, mx, dy1, dx0, dx1)));
    const float DX = fmaxf(fabsf(dx0), fabsf(dx1)), DY = fmaxf(fabsf(dy0), fabsf(dy1));
    const float mag = fabsf(qa) * DX * DX + fabsf(qb) * DX * DY + fabsf(qc) * DY * DY;
    const float thr = -__log2f(255.0f * o) - 1e-5f - 16.0f * 5.9604645e-8f * mag;
    return m >= thr;
}

__device__ __forceinline__ unsigned long long lanes_below(int lane) {
    return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// (one entry more than a chunk, which the last entry's read ahead touches)
struct WaveStage {
    float4 g[kChunk + 1];      // tile-relative mean, qa, qb
    float4 b[kChunk + 1];      // qc, opacity', depth, -
    float4 c[kChunk + 1];      // r, g, b, (int) 1-based position in the tile list
    int4 ps[kChunk];       // 1-based position in the tile list, slot, -, - (16-byte stride like the
                           // records, so one address register serves every per-entry read)
};

// Gathers list entries [j0, j0 + 64) of the tile (clipped to `end`), keeps
// those whose box reaches the quadrant, compacts them in order into `st`;
// returns the number kept.  Wave-uniform.
__device__ __forceinline__ int stage_chunk(const float4* __restrict__ rec, const uint32_t* __restrict__ pair_vals,
                                           uint32_t list0, uint32_t j0, uint32_t end, const PixelCoords& pc,
                                           int lane, WaveStage& st) {
    const uint32_t j = j0 + lane;
    bool hit = false;
    float4 g, r1, r2;
    uint32_t s = 0;
    if (j < end) {
        s = pair_vals[j];
        const float4 r0 = rec[4 * (size_t)s + 0];
        r1 = rec[4 * (size_t)s + 1];
        r2 = rec[4 * (size_t)s + 2];
        const float4 r3 = rec[4 * (size_t)s + 3];
        g = stage_geom(r0, r1, r2, pc.ox, pc.oy);
        hit = box_hits_quadrant(g, r3, pc.qcx, pc.qcy);
    }
    const unsigned long long m = __ballot(hit);
    if (hit) {
        const int d = __popcll(m & lanes_below(lane));
        st.g[d] = g;
        st.b[d] = r1;
        st.c[d] = r2;
        st.ps[d] = make_int4((int)(j - list0) + 1, (int)s, 0, 0);
    }
    __builtin_amdgcn_wave_barrier();
    return __popcll(m);
}

// The compositing backward launches one-wave workgroups, one per (item,
// quadrant): a workgroup of four quadrants holds its LDS and wave slots until
// its slowest quadrant is done, which left half of the slots empty over the
// long lists (their survivors differ from quadrant to quadrant).  Workgroups
// go to the 8 XCDs in turn, so the four quadrants of an item lie 8 apart and
// share an L2, and the items of a run of 8 are rotated from run to run: items
// of a fixed residue are alike (the segments of two-segment lists alternate
// between whole and remainder, which gave every other XCD 45 % more work).
constexpr unsigned kXcds = 8;
struct WaveItem {
    uint32_t item;
    int quad;
};
__device__ __forceinline__ WaveItem wave_item() {
    const uint32_t x = blockIdx.x % kXcds, r = blockIdx.x / kXcds;
    const uint32_t run = r / 4u;
    return WaveItem{run * kXcds + (x + run) % kXcds, (int)(r % 4u)};
}
// workgroups for n items
unsigned wave_grid(unsigned n) { return (n + kXcds - 1) / kXcds * kXcds * 4u; }

// largest i in [0, n] with a[i] <= v (a non-decreasing, a[0] <= v), by one
// wave, 64 probes at a time (wave-uniform arguments)
__device__ __forceinline__ uint32_t last_le_wave(const uint32_t* __restrict__ a, uint32_t n, uint32_t v, int lane) {
    uint32_t lo = 0, hi = n + 1;      // invariant: a[lo] <= v, answer in [lo, hi)
    while (hi - lo > 1) {
        const uint32_t step = (hi - lo + 63) / 64;
        const uint32_t q = lo + (uint32_t)lane * step;
        const bool le = lane == 0 || (q < hi && a[q] <= v);
        const uint32_t L = 63u - (uint32_t)__clzll(__ballot(le));      // lanes 0 .. L hold: a is sorted
        lo = lo + L * step;
        hi = min(hi, lo + step);
    }
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)lo);
}

// work item b of a plan -> launch position: the lists with several segments
// lie in the first info[kPlanLong] positions, each later position is one item
__device__ __forceinline__ uint32_t item_position(const SegPlan& plan, uint32_t b, int lane) {
    const uint32_t k = plan.info[kPlanLong], w = plan.work_off[k];
    return b >= w ? k + (b - w) : last_le_wave(plan.work_off, k, b, lane);
}

// tile at launch position i (the order, when valid, else the position)
__device__ __forceinline__ int order_tile(const uint32_t* __restrict__ tile_order, const ViewTable& vt, uint32_t i) {
    const uint32_t t = tile_order ? tile_order[i] : i;
    return t < (uint32_t)vt.total_tiles ? (int)t : (int)i;
}

// One lane's list entry, loaded a chunk ahead of its use so that the two
// dependent gathers (pair value, then record) overlap the evaluation of the
// previous chunk instead of stalling the wave.  Staging marks the fourth
// record's unused lanes (z, w) as read: registers of a pending load that
// the compiler sees as dead get reused as temporaries, which makes the wave
// wait for the load at once.
struct Gather {
    float4 r0, r1, r2, r3;
    uint32_t slot;
};

constexpr uint32_t kNoSlot = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t load_slot(const uint32_t* __restrict__ pair_vals, uint32_t j, uint32_t end) {
    return j < end ? pair_vals[j] : kNoSlot;
}

__device__ __forceinline__ Gather load_entry(const float4* __restrict__ rec, uint32_t s) {
    Gather g;
    g.slot = s;
    if (s != kNoSlot) {
        g.r0 = rec[4 * (size_t)s + 0];
        g.r1 = rec[4 * (size_t)s + 1];
        g.r2 = rec[4 * (size_t)s + 2];
        g.r3 = rec[4 * (size_t)s + 3];
    } else {
        g.r0 = g.r1 = g.r2 = g.r3 = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
    }
    return g;
}

// box test, ballot and in-order compaction of a gathered chunk into `st`, filled
// up to a multiple of kGroup with entries of opacity 0, which nothing composites;
// pos = the lane's 1-based position in the tile list.  Wave-uniform result.
constexpr int kGroup = 2;
__device__ __forceinline__ int stage_gathered(const Gather& e, int pos, const PixelCoords& pc, int lane,
                                              WaveStage& st) {
    __asm__ volatile("" ::"v"(e.r3.z), "v"(e.r3.w));   // emits no instruction
    const float4 g = stage_geom(e.r0, e.r1, e.r2, pc.ox, pc.oy);
    const bool hit = e.slot != kNoSlot && box_hits_quadrant(g, e.r3, pc.qcx, pc.qcy) &&
                     ellipse_hits_quadrant(g, e.r1, pc.qcx, pc.qcy);
    const unsigned long long m = __ballot(hit);
    if (hit) {
        const int d = __popcll(m & lanes_below(lane));
        st.g[d] = g;
        st.b[d] = make_float4(e.r1.x, e.r1.y, e.r1.z, 0.0f);
        st.c[d] = make_float4(e.r2.x, e.r2.y, e.r2.z, __int_as_float(pos));
    }
    const int n = __popcll(m);
    if (lane >= n && lane < ((n + kGroup - 1) & ~(kGroup - 1)))
        st.g[lane] = st.b[lane] = st.c[lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    __builtin_amdgcn_wave_barrier();
    return n;
}

// segmented forward: stop_seg value of a pixel still compositing after the head
constexpr int32_t kSegAlive = 0x7fffffff;

// positions whose terms the forward adds up at a time
constexpr int kSumPart = 512;

// One wave composites quadrant `quad` of `tile` (staging in its LDS slice
// `st`) and writes its pixels: the whole list, front to back.  With
// head_stop (the tile's stop_seg row; a list the plan segments) only the
// head, the first head_len positions: pixels that stop there (or whose list
// ends there) get their outputs and stop_seg = -1, the others their state
// after it (rgb without background, depth, T, last) and stop_seg =
// kSegAlive.  The head also writes the backward's states of its segments from
// 1 on (seg_len positions; head_states: the tile's first stored state): T_seg =
// T_end / T_start and C_seg = C / T_start, C the segment's own part of the sum --
// its composite with T restarted at 1.  So the sums restart at each segment and
// the parts are added up: the difference of a running sum at the segment's ends
// would carry rounding at the size of the whole sum, which is large beside a deep
// segment's part (4096 Gaussians at 160x120, several segments of 128 to a head:
// opacity and mean gradients twice as far from float64, and the image 1.3 times).
// Every walk adds up parts of at most kSumPart positions, whose length bounds the
// rounding of a sum: long lists in segments of 2048 came out 1.4 times as far from
// float64 as in segments of 512.
__device__ __forceinline__ void render_fwd_quadrant(const float4* __restrict__ rec,
                                                    const uint32_t* __restrict__ pair_vals,
                                                    const uint2* __restrict__ ranges, const ViewTable& vt,
                                                    const OptK& opt, int tile, int quad, int lane, WaveStage& st,
                                                    float* __restrict__ rgb, float* __restrict__ depth,
                                                    float* __restrict__ alpha_out, float* __restrict__ T_out,
                                                    int32_t* __restrict__ last_out,
                                                    int32_t* __restrict__ head_stop = nullptr,
                                                    float* __restrict__ head_states = nullptr,
                                                    uint32_t seg_len = kSegLen, uint32_t head_len = kHeadLen) {
    const PixelCoords pc = pixel_coords(vt, tile, quad, lane);
    const uint2 rg = ranges[tile];
    const uint32_t end = head_stop ? min(rg.x + head_len, rg.y) : rg.y;

    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, D = 0.0f;
    int last = 0;
    bool alive = pc.inside;
    // T at the start of the current segment, its (C, D) before the current part, and the earlier ones'
    float sT = 1.0f, s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, sD = 0.0f, t0 = 0.0f, t1 = 0.0f, t2 = 0.0f, tD = 0.0f;
    const uint32_t part = min(seg_len, (uint32_t)kSumPart);
    int seg = 0;
    const int px = pc.ly * kTile + pc.lx;
    auto seg_state = [&]() {      // state of segment `seg` >= 1 from its start to now
        float* o = head_states + (size_t)(seg - 1) * kSegFields * 256;
        const float inv = 1.0f / sT;
        o[0 * 256 + px] = T * inv;
        o[1 * 256 + px] = s0 * inv;
        o[2 * 256 + px] = s1 * inv;
        o[3 * 256 + px] = s2 * inv;
        o[4 * 256 + px] = sD * inv;
    };
    auto end_part = [&]() {
        s0 += c0;
        s1 += c1;
        s2 += c2;
        sD += D;
        c0 = c1 = c2 = D = 0.0f;
    };
    Gather cur = load_entry(rec, load_slot(pair_vals, rg.x + lane, end));
    uint32_t s_next = load_slot(pair_vals, rg.x + kChunk + lane, end);
    for (uint32_t j0 = rg.x; j0 < end; j0 += kChunk) {
        if (j0 != rg.x && ((j0 - rg.x) & (part - 1u)) == 0) {
            end_part();
            if (((j0 - rg.x) & (seg_len - 1u)) == 0) {
                if (head_states && seg >= 1) seg_state();
                ++seg;
                sT = T;
                t0 += s0;
                t1 += s1;
                t2 += s2;
                tD += sD;
                s0 = s1 = s2 = sD = 0.0f;
            }
        }
        if (__ballot(alive) == 0) break;     // every pixel of the quadrant has stopped
        const int n = stage_gathered(cur, (int)(j0 - rg.x) + lane + 1, pc, lane, st);
        cur = load_entry(rec, s_next);                                   // next chunk's records
        s_next = load_slot(pair_vals, j0 + 2 * kChunk + lane, end);      // and the one after's slots
        // entry k + 1 is read from LDS while entry k is evaluated, kGroup entries
        // from one address and under one bound: 1M Gaussians 237 -> 221 us, 6M
        // 170 -> 157 (groups of 4 spill)
        float4 an = st.g[0], bn = st.b[0], cn = st.c[0];
        for (int k = 0; k < n; k += kGroup) {
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
                const float4 a = an, b = bn, c = cn;
                an = st.g[k + u + 1];
                bn = st.b[k + u + 1];
                cn = st.c[k + u + 1];
                const Eval e = eval_entry(a, b, pc.fpx, pc.fpy);
                const float Tn = T * (1.0f - e.alpha);
                const bool keep = alive && e.keep;
                const bool stop = keep && Tn < kTMin;
                const bool use = keep && !stop;
                const float w = use ? e.alpha * T : 0.0f;
                c0 = fmaf(c.x, w, c0);
                c1 = fmaf(c.y, w, c1);
                c2 = fmaf(c.z, w, c2);
                D = fmaf(b.z, w, D);
                T = use ? Tn : T;
                last = use ? __float_as_int(c.w) : last;
                alive = alive && !stop;
            }
        }
        __builtin_amdgcn_wave_barrier();     // the chunk is consumed before the next one is staged
    }
    end_part();
    if (head_states && seg >= 1) seg_state();
    c0 = t0 + s0;
    c1 = t1 + s1;
    c2 = t2 + s2;
    D = tD + sD;
    if (!pc.inside) return;
    const int64_t p = pc.pix;
    const bool more = head_stop && alive && end < rg.y;    // compositing continues after the head
    if (head_stop) head_stop[px] = more ? kSegAlive : -1;
    rgb[3 * p + 0] = more ? c0 : fmaf(T, opt.bg[0], c0);
    rgb[3 * p + 1] = more ? c1 : fmaf(T, opt.bg[1], c1);
    rgb[3 * p + 2] = more ? c2 : fmaf(T, opt.bg[2], c2);
    depth[p] = D;
    if (!more) alpha_out[p] = 1.0f - T;
    T_out[p] = T;
    last_out[p] = last;
}

// Segmented forward, pass 2: one wave walks segment `seg` past the head
// (list positions [seg S, (seg + 1) S), S = seg_len) of a long list for the
// pixels of its quadrant still compositing after the head (`on`),
// and keeps, over the entries that pass the alpha test, the segment's
// state with T restarted at 1: T_seg = prod (1 - alpha), C_seg = sum c
// alpha T_local (colour and depth) and the position of its last such entry
// -- as if no pixel stopped in the segment -- in its stored-state row
// (planes T, r, g, b, depth, last; the other pixels get the empty state).
// A pixel whose T_local falls below T_min is certain to stop in this
// segment or an earlier one (T before it is at most 1); it is left there
// (the fold then stops in or before this segment, whose exact walk pass 4
// redoes), and the wave stops when all its pixels are.
__device__ __forceinline__ void render_fwd_segment(const float4* __restrict__ rec,
                                                   const uint32_t* __restrict__ pair_vals, const uint2 rg,
                                                   const PixelCoords& pc, bool on, int seg, uint32_t seg_len, int lane,
                                                   WaveStage& st, float* __restrict__ state_row) {
    const uint32_t lo = rg.x + (uint32_t)seg * seg_len, hi = min(lo + seg_len, rg.y);
    float Tl = 1.0f, l0 = 0.0f, l1 = 0.0f, l2 = 0.0f, Dl = 0.0f;
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, sD = 0.0f;      // earlier parts
    int last = 0;
    Gather cur = load_entry(rec, load_slot(pair_vals, lo + lane, hi));
    uint32_t s_next = load_slot(pair_vals, lo + kChunk + lane, hi);
    for (uint32_t j0 = lo; j0 < hi; j0 += kChunk) {
        if (__ballot(on) == 0) break;
        if (j0 != lo && ((j0 - lo) & (kSumPart - 1u)) == 0) {
            s0 += l0;
            s1 += l1;
            s2 += l2;
            sD += Dl;
            l0 = l1 = l2 = Dl = 0.0f;
        }
        const int n = stage_gathered(cur, (int)(j0 - rg.x) + lane + 1, pc, lane, st);
        cur = load_entry(rec, s_next);
        s_next = load_slot(pair_vals, j0 + 2 * kChunk + lane, hi);
        for (int k = 0; k < n; k += kGroup) {
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
                const float4 a = st.g[k + u], b = st.b[k + u], c = st.c[k + u];
                const Eval e = eval_entry(a, b, pc.fpx, pc.fpy);
                const bool use = on && e.keep;
                const float w = use ? e.alpha * Tl : 0.0f;
                l0 = fmaf(c.x, w, l0);
                l1 = fmaf(c.y, w, l1);
                l2 = fmaf(c.z, w, l2);
                Dl = fmaf(b.z, w, Dl);
                Tl = use ? Tl * (1.0f - e.alpha) : Tl;
                last = use ? __float_as_int(c.w) : last;
            }
        }
        on = on && Tl >= kTMin;
        __builtin_amdgcn_wave_barrier();
    }
    const int px = pc.ly * kTile + pc.lx;
    state_row[0 * 256 + px] = Tl;
    state_row[1 * 256 + px] = s0 + l0;
    state_row[2 * 256 + px] = s1 + l1;
    state_row[3 * 256 + px] = s2 + l2;
    state_row[4 * 256 + px] = sD + Dl;
    reinterpret_cast<int32_t*>(state_row)[5 * 256 + px] = last;
}

// stored segment b of a plan -> launch position, segment (>= 1), count
struct SegItem {
    uint32_t i;
    int seg, nseg;
};
__device__ __forceinline__ SegItem stored_seg(const SegPlan& plan, uint32_t b, int lane) {
    SegItem it;
    it.i = last_le_wave(plan.state_off, plan.info[kPlanLong], b, lane);      // no states past it
    it.seg = (int)(b - plan.state_off[it.i]) + 1;
    it.nseg = (int)(plan.work_off[it.i + 1] - plan.work_off[it.i]);
    return it;
}

// One workgroup per tile, in launch order.  With a segment plan, the lists
// it segments composite their head only (pass 1 of the segmented forward).
// (256, 7): at most 72 VGPRs, 7 waves per SIMD; 10 registers spilled, most of them
// the sums that only the ends of parts and segments touch.
__global__ __launch_bounds__(256, 7) void k_render_fwd(const float4* __restrict__ rec,
                                                    const uint32_t* __restrict__ pair_vals,
                                                    const uint2* __restrict__ ranges,
                                                    const uint32_t* __restrict__ tile_order, ViewTable vt, OptK opt,
                                                    float* __restrict__ rgb, float* __restrict__ depth,
                                                    float* __restrict__ alpha_out, float* __restrict__ T_out,
                                                    int32_t* __restrict__ last_out, SegPlan plan) {
    __shared__ WaveStage stage[kWaves];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int tile = launch_tile(tile_order, vt);
    int32_t* head_stop = nullptr;
    float* head_states = nullptr;
    uint32_t seg_len = kSegLen, head_len = kHeadLen;
    if (plan.work_off) {
        const uint32_t i = blockIdx.x;
        if (plan.work_off[i + 1] - plan.work_off[i] > 1u) {
            seg_len = plan.info[kPlanLen];
            head_len = plan.info[kPlanHead] * seg_len;
            head_stop = plan.stop_seg + (size_t)tile * 256;
            head_states = plan.state + (size_t)plan.state_off[i] * kSegFields * 256;
        }
    }
    render_fwd_quadrant(rec, pair_vals, ranges, vt, opt, tile, wave, lane, stage[wave], rgb, depth, alpha_out, T_out,
                        last_out, head_stop, head_states, seg_len, head_len);
}

// Pass 2, one workgroup per stored segment: the segment's state for the
// pixels still compositing after the head (a quadrant with none exits).
// (256, 7): at most 72 VGPRs, 7 waves per SIMD, no spills.
__global__ __launch_bounds__(256, 7) void k_fwd_segments(const float4* __restrict__ rec,
                                                      const uint32_t* __restrict__ pair_vals,
                                                      const uint2* __restrict__ ranges,
                                                      const uint32_t* __restrict__ tile_order, ViewTable vt,
                                                      SegPlan plan) {
    __shared__ WaveStage stage[kWaves];
    const uint32_t b = blockIdx.x;
    if (b >= plan.state_off[plan.n_tiles]) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const SegItem it = stored_seg(plan, b, lane);
    if (it.seg < (int)plan.info[kPlanHead]) return;        // the head's segments
    const int tile = order_tile(tile_order, vt, it.i);
    const PixelCoords pc = pixel_coords(vt, tile, wave, lane);
    const bool on = pc.inside && plan.stop_seg[(size_t)tile * 256 + pc.ly * kTile + pc.lx] == kSegAlive;
    if (__ballot(on) == 0) return;
    render_fwd_segment(rec, pair_vals, ranges[tile], pc, on, it.seg, plan.info[kPlanLen], lane, stage[wave],
                       plan.state + (size_t)b * kSegFields * 256);
}

// Pass 3, one thread per pixel still compositing after the head of a
// segmented list: fold the segments after it front to back (C += T C_seg,
// T *= T_seg).  T only decreases along the list, so the pixel stops inside
// segment j exactly when T T_seg_j < T_min; then its state before segment j
// is left in the outputs and stop_seg = j for pass 4.  Otherwise the
// outputs are final and stop_seg = -1.
__global__ __launch_bounds__(256) void k_fwd_combine(const uint32_t* __restrict__ tile_order, ViewTable vt,
                                                     OptK opt, SegPlan plan, float* __restrict__ rgb,
                                                     float* __restrict__ depth, float* __restrict__ alpha_out,
                                                     float* __restrict__ T_out, int32_t* __restrict__ last_out) {
    const uint32_t i = blockIdx.x;
    const int nseg = (int)(plan.work_off[i + 1] - plan.work_off[i]);
    if (nseg <= 1) return;
    const int tile = order_tile(tile_order, vt, i);
    const PixelCoords pc = pixel_coords(vt, tile, threadIdx.x >> 6, threadIdx.x & 63);
    const int px = pc.ly * kTile + pc.lx;
    int32_t* stop_row = plan.stop_seg + (size_t)tile * 256;
    if (!pc.inside || stop_row[px] != kSegAlive) return;
    const int64_t p = pc.pix;
    float T = T_out[p], c0 = rgb[3 * p + 0], c1 = rgb[3 * p + 1], c2 = rgb[3 * p + 2], D = depth[p];
    int last = last_out[p];
    int stop = -1;
    const uint32_t st0 = plan.state_off[i];
    // kFold segments' states are read together, so that the fold waits for
    // one round of loads per kFold of them
    constexpr int kFold = 4;
    for (int j0 = (int)plan.info[kPlanHead]; j0 < nseg && stop < 0; j0 += kFold) {
        float s[kFold][5];
        int sl[kFold];
#pragma unroll
        for (int u = 0; u < kFold; ++u) {
            const int j = min(j0 + u, nseg - 1);
            const float* r = plan.state + (size_t)(st0 + (uint32_t)(j - 1)) * kSegFields * 256;
#pragma unroll
            for (int q = 0; q < 5; ++q) s[u][q] = r[q * 256 + px];
            sl[u] = reinterpret_cast<const int32_t*>(r)[5 * 256 + px];
        }
#pragma unroll
        for (int u = 0; u < kFold; ++u) {
            if (j0 + u >= nseg || stop >= 0) continue;
            if (T * s[u][0] < kTMin) {
                stop = j0 + u;
                continue;
            }
            c0 = fmaf(T, s[u][1], c0);
            c1 = fmaf(T, s[u][2], c1);
            c2 = fmaf(T, s[u][3], c2);
            D = fmaf(T, s[u][4], D);
            T *= s[u][0];
            last = sl[u] > 0 ? sl[u] : last;
        }
    }
    stop_row[px] = stop;
    if (stop < 0) {
        rgb[3 * p + 0] = fmaf(T, opt.bg[0], c0);
        rgb[3 * p + 1] = fmaf(T, opt.bg[1], c1);
        rgb[3 * p + 2] = fmaf(T, opt.bg[2], c2);
        alpha_out[p] = 1.0f - T;
    } else {
        rgb[3 * p + 0] = c0;
        rgb[3 * p + 1] = c1;
        rgb[3 * p + 2] = c2;
    }
    depth[p] = D;
    T_out[p] = T;
    last_out[p] = last;
}

// Pass 4, one workgroup per stored segment: the pixels that stop in this
// segment walk it again from their state before it, with the stop rule,
// T = T_start T_local and T_local recomputed as in pass 2 (so the pixel
// stops here, at the latest at the segment's last entry); they write their
// final outputs and the segment's state over the entries they composited
// (the state the backward folds).  (256, 7): 7 waves per SIMD, no spills.
__global__ __launch_bounds__(256, 7) void k_fwd_fix(const float4* __restrict__ rec,
                                                 const uint32_t* __restrict__ pair_vals,
                                                 const uint2* __restrict__ ranges,
                                                 const uint32_t* __restrict__ tile_order, ViewTable vt, OptK opt,
                                                 SegPlan plan, float* __restrict__ rgb, float* __restrict__ depth,
                                                 float* __restrict__ alpha_out, float* __restrict__ T_out,
                                                 int32_t* __restrict__ last_out) {
    __shared__ WaveStage stage[kWaves];
    const uint32_t b = blockIdx.x;
    if (b >= plan.state_off[plan.n_tiles]) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const SegItem it = stored_seg(plan, b, lane);
    const int tile = order_tile(tile_order, vt, it.i);
    const PixelCoords pc = pixel_coords(vt, tile, wave, lane);
    const int px = pc.ly * kTile + pc.lx;
    bool alive = pc.inside && plan.stop_seg[(size_t)tile * 256 + px] == it.seg;
    const bool mine = alive;
    if (__ballot(alive) == 0) return;      // no pixel of the quadrant stops here
    WaveStage& st = stage[wave];
    const uint2 rg = ranges[tile];
    float Ts = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, D0 = 0.0f;
    int last = 0;
    if (mine) {
        const int64_t p = pc.pix;
        Ts = T_out[p];
        C0 = rgb[3 * p + 0];
        C1 = rgb[3 * p + 1];
        C2 = rgb[3 * p + 2];
        D0 = depth[p];
        last = last_out[p];
    }
    const uint32_t seg_len = plan.info[kPlanLen], lo = rg.x + (uint32_t)it.seg * seg_len, hi = min(lo + seg_len, rg.y);
    float Tl = 1.0f, l0 = 0.0f, l1 = 0.0f, l2 = 0.0f, Dl = 0.0f;
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, sD = 0.0f;      // earlier parts
    Gather cur = load_entry(rec, load_slot(pair_vals, lo + lane, hi));
    uint32_t s_next = load_slot(pair_vals, lo + kChunk + lane, hi);
    for (uint32_t j0 = lo; j0 < hi; j0 += kChunk) {
        if (__ballot(alive) == 0) break;
        if (j0 != lo && ((j0 - lo) & (kSumPart - 1u)) == 0) {
            s0 += l0;
            s1 += l1;
            s2 += l2;
            sD += Dl;
            l0 = l1 = l2 = Dl = 0.0f;
        }
        const int n = stage_gathered(cur, (int)(j0 - rg.x) + lane + 1, pc, lane, st);
        cur = load_entry(rec, s_next);
        s_next = load_slot(pair_vals, j0 + 2 * kChunk + lane, hi);
        for (int k = 0; k < n; k += kGroup) {
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
                const float4 a = st.g[k + u], bb = st.b[k + u], c = st.c[k + u];
                const Eval e = eval_entry(a, bb, pc.fpx, pc.fpy);
                const bool keep = alive && e.keep;
                const float Tln = Tl * (1.0f - e.alpha);
                const bool stop = keep && Ts * Tln < kTMin;
                const bool use = keep && !stop;
                const float w = use ? e.alpha * Tl : 0.0f;
                l0 = fmaf(c.x, w, l0);
                l1 = fmaf(c.y, w, l1);
                l2 = fmaf(c.z, w, l2);
                Dl = fmaf(bb.z, w, Dl);
                Tl = use ? Tln : Tl;
                last = use ? __float_as_int(c.w) : last;
                alive = alive && !stop;
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (!mine) return;
    l0 += s0;
    l1 += s1;
    l2 += s2;
    Dl += sD;
    const int64_t p = pc.pix;
    const float T = Ts * Tl;
    rgb[3 * p + 0] = fmaf(T, opt.bg[0], fmaf(Ts, l0, C0));
    rgb[3 * p + 1] = fmaf(T, opt.bg[1], fmaf(Ts, l1, C1));
    rgb[3 * p + 2] = fmaf(T, opt.bg[2], fmaf(Ts, l2, C2));
    depth[p] = fmaf(Ts, Dl, D0);
    alpha_out[p] = 1.0f - T;
    T_out[p] = T;
    last_out[p] = last;
    float* r = plan.state + (size_t)b * kSegFields * 256;
    r[0 * 256 + px] = Tl;
    r[1 * 256 + px] = l0;
    r[2 * 256 + px] = l1;
    r[3 * 256 + px] = l2;
    r[4 * 256 + px] = Dl;
}

// Persistent compositing: a fixed grid whose workgroups take tiles in launch
// order (longest lists first) from a counter until every tile is taken; the
// four waves composite the tile's quadrants, as in the one-tile-per-workgroup
// launch, so a tile's records are fetched into one compute unit's cache.  The
// next tile is taken while the current one composites.  A grid smaller than
// the device leaves compute units to work on other streams.
__global__ __launch_bounds__(256) void k_render_fwd_persistent(const float4* __restrict__ rec,
                                                               const uint32_t* __restrict__ pair_vals,
                                                               const uint2* __restrict__ ranges,
                                                               const uint32_t* __restrict__ tile_order, ViewTable vt,
                                                               OptK opt, float* __restrict__ rgb,
                                                               float* __restrict__ depth,
                                                               float* __restrict__ alpha_out,
                                                               float* __restrict__ T_out,
                                                               int32_t* __restrict__ last_out,
                                                               uint32_t* __restrict__ work) {
    __shared__ WaveStage stage[kWaves];
    __shared__ uint32_t s_item[2];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t n_items = (uint32_t)vt.total_tiles;
    if (threadIdx.x == 0) s_item[0] = atomicAdd(work, 1u);
    __syncthreads();
    int k = 0;
    uint32_t item = s_item[0];
    // every wave of the workgroup reads the same item, so all leave together
    while (item < n_items) {
        if (threadIdx.x == 0) s_item[k ^ 1] = atomicAdd(work, 1u);
        render_fwd_quadrant(rec, pair_vals, ranges, vt, opt, order_tile(tile_order, vt, item), wave, lane,
                            stage[wave], rgb, depth, alpha_out, T_out, last_out);
        __syncthreads();     // the next item is in LDS; its slot is rewritten only after the next barrier
        k ^= 1;
        item = s_item[k];
    }
}

// Per pixel: the number of list entries compositing must evaluate -- those
// whose box contains the pixel centre, up to and including the one that
// stops the pixel.  The unit of work of compositing; measurement only.
__global__ __launch_bounds__(256) void k_render_count(const float4* __restrict__ rec,
                                                      const uint32_t* __restrict__ pair_vals,
                                                      const uint2* __restrict__ ranges,
                                                      const uint32_t* __restrict__ tile_order, ViewTable vt,
                                                      int32_t* __restrict__ n_eval) {
    __shared__ WaveStage stage[kWaves];
    __shared__ float2 sbox[kWaves][kChunk];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int tile = launch_tile(tile_order, vt);
    const PixelCoords pc = pixel_coords(vt, tile, wave, lane);
    WaveStage& st = stage[wave];
    const uint2 rg = ranges[tile];
    float T = 1.0f;
    int count = 0, count_last = 0;
    bool alive = pc.inside;
    for (uint32_t j0 = rg.x; j0 < rg.y; j0 += kChunk) {
        if (__ballot(alive) == 0) break;
        const int n = stage_chunk(rec, pair_vals, rg.x, j0, rg.y, pc, lane, st);
        if (lane < n) {
            const float4 r3 = rec[4 * (size_t)(uint32_t)st.ps[lane].y + 3];
            sbox[wave][lane] = make_float2(r3.x, r3.y);
        }
        __builtin_amdgcn_wave_barrier();
        for (int k = 0; k < n; ++k) {
            const float4 a = st.g[k], b = st.b[k];
            const float2 h = sbox[wave][k];
            const bool covers = fabsf(pc.fpx - a.x) <= h.x && fabsf(pc.fpy - a.y) <= h.y;
            const Eval e = eval_entry(a, b, pc.fpx, pc.fpy);
            const float Tn = T * (1.0f - e.alpha);
            const bool keep = alive && e.keep;
            const bool stop = keep && Tn < kTMin;
            count += (alive && covers) ? 1 : 0;
            count_last = (keep && !stop) ? count : count_last;
            T = (keep && !stop) ? Tn : T;
            alive = alive && !stop;
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (pc.inside) reinterpret_cast<int2*>(n_eval)[pc.pix] = make_int2(count, count_last);
}

constexpr int kG2 = GS_GRAD2D_FLOATS;   // per-slot 2D gradient fields

// One wave's LDS of the backward: the chunk's surviving entries (their
// records overwritten by their gradient sums once reduced), the per-pixel
// values of a batch of kBatch entries, and the pixels' upstream gradients.
constexpr int kBatch = 8;
constexpr int kQW = 68;                 // an entry's row: dp of 64 pixels, padding, w of 64 pixels
constexpr int kQRow = 132;              // the next entry starts 4 banks further
template <bool kAbs>
struct alignas(16) BwdStage {
    float4 r[kChunk][3];       // mean, qa, qb | qc, opacity', depth, slot (bits) | r, g, b, position (1-based, bits)
    float q[kBatch * kQRow];   // [entry of the batch][dp, w][pixel]
    float4 up[65];             // upstream gradients by pixel, one further from y = 4 on (banks)
    uint32_t slot[kAbs ? kChunk : 1];       // slots of the reduced rows; in word 10 of a row of 10 fields
};

// load_entry and stage_gathered for the backward; only the used half of the
// fourth record is loaded
struct GatherBwd {
    float4 r0, r1, r2;
    float2 r3;
    uint32_t slot;
};
__device__ __forceinline__ GatherBwd load_entry_bwd(const float4* __restrict__ rec, uint32_t s) {
    GatherBwd g;
    g.slot = s;
    if (s != kNoSlot) {
        g.r0 = rec[4 * (size_t)s + 0];
        g.r1 = rec[4 * (size_t)s + 1];
        g.r2 = rec[4 * (size_t)s + 2];
        g.r3 = *reinterpret_cast<const float2*>(rec + 4 * (size_t)s + 3);
    } else {
        g.r0 = g.r1 = g.r2 = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
        g.r3 = make_float2(0.0f, 0.0f);
    }
    return g;
}
template <class Stage>
__device__ __forceinline__ int stage_gathered_bwd(const GatherBwd& e, int pos, const PixelCoords& pc, int lane,
                                                  Stage& st) {
    const float4 g = stage_geom(e.r0, e.r1, e.r2, pc.ox, pc.oy);
    const bool hit = e.slot != kNoSlot &&
                     box_hits_quadrant(g, make_float4(e.r3.x, e.r3.y, 0.0f, 0.0f), pc.qcx, pc.qcy) &&
                     ellipse_hits_quadrant(g, e.r1, pc.qcx, pc.qcy);
    const unsigned long long m = __ballot(hit);
    if (hit) {
        const int d = __popcll(m & lanes_below(lane));
        st.r[d][0] = g;
        st.r[d][1] = make_float4(e.r1.x, e.r1.y, e.r1.z, __uint_as_float(e.slot));
        st.r[d][2] = make_float4(e.r2.x, e.r2.y, e.r2.z, __int_as_float(pos));
    }
    __builtin_amdgcn_wave_barrier();
    return __popcll(m);
}

// Backward: each wave walks its quadrant's list back to front from the
// deepest `last` of its pixels, in chunks staged and culled as in the
// forward.  The colour and depth behind an entry enter the gradient only
// through their dot product with the pixel's upstream gradient, so the walk
// carries that one scalar, S = g_rgb . R_rgb + g_depth R_depth, instead of R.
//
// The 2D gradients of an entry are sums over the quadrant's 64 pixels of two
// per-pixel values -- dp = dL/d(exponent) and w = alpha T -- times factors
// that depend on the pixel and the entry's mean alone: dp times 1, dx, dy,
// dx^2, dx dy, dy^2 and w times the pixel's upstream gradient.  The walk only
// leaves dp and w in LDS; every 8 entries they are read back transposed, lane
// (y, entry) taking the 8 pixels of row y, whose dp, dp dx and dp dx^2 it sums in
// registers; dy is constant in a row.  Three exchanges over the 8 rows finish the
// sums.  That is about 14 VALU instructions per entry; a sum of each field over the
// wave by lane exchanges takes 30 and its products 14 more (6M Gaussians, 1080p,
// bound by VALU issue: 0.60 ms, 0.56 now).  (Moments about the quadrant's centre,
// shifted to the mean after the sum, save two more instructions and 1 % of the
// time, but cancel: for Gaussians of pixel size near a quadrant's corner dp dx^2
// came out with 26 times the rounding error of its products.)  The FP32 matrix
// instructions were measured too: they share the vector units' time (an fma beside
// v_mfma_f32_16x16x4_f32 adds its own) and fill a third of a product here, 27 ns
// per entry against 14.
// The AbsGS sums (kAbs) come from the same rows: |dp| |2 qa dx + qb dy| and
// |dp| |qb dx + 2 qc dy| per pixel.
//
// The sums overwrite staged records the walk has passed; after the chunk the
// wave adds them to the per-slot rows, one float atomic per nonzero field.
//
// T is divided back by 1 - alpha an entry at a time, with the reciprocal's estimate,
// whose error (up to an ulp, alike for alike alphas) adds up over the walk.  In
// segments longer than kSegLen (kLong) a Newton step takes it to half an ulp either
// way: two instructions an entry, with which walks of 2048 are nearer float64 than
// walks of 512 with the estimate (without, up to 4 times as far; 12M Gaussians in
// eight views 5.86 -> 5.95 ms).
// (64, 5): 96 VGPRs without spills, five waves per SIMD; 19 workgroups share a
// compute unit's LDS.
template <bool kAbs, bool kLong>
__global__ __launch_bounds__(64, 5) void k_render_bwd(const float4* __restrict__ rec,
                                                   const uint32_t* __restrict__ pair_vals,
                                                   const uint2* __restrict__ ranges,
                                                   const uint32_t* __restrict__ tile_order, ViewTable vt, OptK opt,
                                                   const float* __restrict__ T_final,
                                                   const int32_t* __restrict__ last_in,
                                                   const float* __restrict__ d_rgb, const float* __restrict__ d_depth,
                                                   const float* __restrict__ d_alpha, float* __restrict__ grad2d,
                                                   SegPlan plan) {
    __shared__ BwdStage<kAbs> st;
    const int lane = threadIdx.x;
    const WaveItem wi = wave_item();
    const uint32_t b = wi.item;
    int tile, seg = 0, nseg = 1;
    uint32_t st0 = 0;
    if (plan.work_off) {
        // work item -> (launch position, segment)
        if (b >= plan.work_off[plan.n_tiles]) return;
        const uint32_t i = item_position(plan, b, lane);
        seg = (int)(b - plan.work_off[i]);
        nseg = (int)(plan.work_off[i + 1] - plan.work_off[i]);
        st0 = plan.state_off[i];
        tile = order_tile(tile_order, vt, i);
    } else {
        if (b >= (uint32_t)vt.total_tiles) return;
        tile = order_tile(tile_order, vt, b);
    }
    const PixelCoords pc = pixel_coords(vt, tile, wi.quad, lane);
    const uint2 rg = ranges[tile];

    float T = 1.0f, gC0 = 0.0f, gC1 = 0.0f, gC2 = 0.0f, gD = 0.0f, gA = 0.0f;
    int last = 0;
    if (pc.inside) {
        const int64_t p = pc.pix;
        T = T_final[p];
        last = last_in[p];
        if (d_rgb) {
            gC0 = d_rgb[3 * p + 0];
            gC1 = d_rgb[3 * p + 1];
            gC2 = d_rgb[3 * p + 2];
        }
        if (d_depth) gD = d_depth[p];
        if (d_alpha) gA = d_alpha[p];
    }
    int maxlast = last;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) maxlast = max(maxlast, __shfl_xor(maxlast, off, 64));

    // R = remaining colour behind the entry divided by T after it (starts at
    // bg); the walk keeps S = g . R
    float S = fmaf(gC0, opt.bg[0], fmaf(gC1, opt.bg[1], gC2 * opt.bg[2])), Q = 1.0f;

    // A segmented list: this workgroup walks segment `seg` (positions
    // (seg S, (seg + 1) S]); the state behind it comes from folding the later
    // segments' transmittance and local colour, written by the forward or
    // k_seg_prepass: R <- C_j + T_j R (so S <- g . C_j + T_j S), T <- T / T_j,
    // Q <- Q T_j (segments starting at or after the pixel's last composited
    // entry are the identity).
    int lo = 0, hi = maxlast;
    if (nseg > 1) {
        const int px = pc.ly * kTile + pc.lx, seg_len = (int)plan.info[kPlanLen];
        for (int j = nseg - 1; j > seg; --j) {
            if (j * seg_len >= last) continue;
            const float* sj = plan.state + (size_t)(st0 + (uint32_t)(j - 1)) * kSegFields * 256;
            const float Ts = sj[0 * 256 + px];
            const float gcs = fmaf(gC0, sj[1 * 256 + px],
                                   fmaf(gC1, sj[2 * 256 + px], fmaf(gC2, sj[3 * 256 + px], gD * sj[4 * 256 + px])));
            S = fmaf(Ts, S, gcs);
            T = T / Ts;
            Q = Q * Ts;
        }
        lo = seg * seg_len;
        hi = min(lo + seg_len, maxlast);
    }
    if (hi <= lo) return;

    // Transposed: lane (y, j) takes row y of the quadrant of entry j of a
    // batch.  y is spread over lane bits 5, 4 (lane swaps) and 0 (quad
    // permutation); rows y and y + 4 of 8 entries, 16 consecutive lanes, then
    // read from all 64 banks.
    const int ty = (lane >> 4) | ((lane & 1) << 2), tj = (lane >> 1) & 7;
    const float Yc = pc.qcy + ((float)ty - 3.5f);
    st.up[lane + (lane >> 5)] = make_float4(gC0, gC1, gC2, gD);
    __builtin_amdgcn_wave_barrier();
    const float4* up = &st.up[8 * ty + (ty >> 2)];      // upstream gradients of the row's pixels

    // Reduces the batch's nb entries: staged index of entry e in byte e of
    // `ks`; their gradient sums go to the staged rows top - e, which the walk
    // has passed already (top - e is not below the entry's own row).
    constexpr int kFields = kAbs ? kG2 : 10;
    auto reduce = [&](int nb, uint64_t ks, int top) {
        __builtin_amdgcn_wave_barrier();
        const int k = (int)((ks >> (8 * tj)) & 63u);
        const float4 a = st.r[k][0], b = st.r[k][1];
        const float* q = &st.q[tj * kQRow + 8 * ty];
        const float4 p0 = *reinterpret_cast<const float4*>(q), p1 = *reinterpret_cast<const float4*>(q + 4);
        const float pv[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
        // the mean from the quadrant's left edge: exact where a pixel may lie near it
        const float mx = a.x - (pc.qcx - 4.0f), dy = Yc - a.y;
        float m0 = 0.0f, sx = 0.0f, sxx = 0.0f;      // sums of dp, dp dx, dp dx^2
#pragma unroll
        for (int x = 0; x < 8; ++x) {
            const float dx = ((float)x + 0.5f) - mx, px = pv[x] * dx;
            m0 += pv[x];
            sx += px;
            sxx = fmaf(px, dx, sxx);
        }
        const float sy = dy * m0;
        float v[12];
        v[0] = -kLn2 * fmaf(a.z + a.z, sx, a.w * sy);
        v[1] = -kLn2 * fmaf(a.w, sx, (b.x + b.x) * sy);
        v[2] = -0.5f * sxx;
        v[3] = -dy * sx;
        v[4] = -0.5f * dy * sy;
        v[5] = m0 * __builtin_amdgcn_rcpf(b.y);                 // dp = dL/d opacity' opacity'
        if (kAbs) {
            const float qb = 0.5f * a.w, hx0 = qb * dy, hy0 = b.x * dy;
            float ax = 0.0f, ay = 0.0f;
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const float dx = ((float)x + 0.5f) - mx;
                ax = fmaf(fabsf(pv[x]), fabsf(fmaf(a.z, dx, hx0)), ax);
                ay = fmaf(fabsf(pv[x]), fabsf(fmaf(qb, dx, hy0)), ay);
            }
            v[10] = (2.0f * kLn2) * ax;
            v[11] = (2.0f * kLn2) * ay;
        }
        {
            const float4 w0 = *reinterpret_cast<const float4*>(q + kQW);
            const float4 w1 = *reinterpret_cast<const float4*>(q + kQW + 4);
            const float wv[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
            v[6] = v[7] = v[8] = v[9] = 0.0f;
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const float4 u = up[x];
                v[6] = fmaf(u.x, wv[x], v[6]);
                v[7] = fmaf(u.y, wv[x], v[7]);
                v[8] = fmaf(u.z, wv[x], v[8]);
                v[9] = fmaf(u.w, wv[x], v[9]);
            }
        }
        // sums over the rows: the lane halves swap half of the fields, the
        // rows of 16 lanes half of what is left, lane pairs add up
        float h[6], out[3];
#pragma unroll
        for (int i = 0; i < kFields / 2; ++i) {
            const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + kFields / 2]),
                                                            false, false);
            h[i] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
        }
        if (!kAbs) h[5] = 0.0f;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(h[2 * i]), __float_as_uint(h[2 * i + 1]),
                                                            false, false);
            const float x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
            out[i] = x + __builtin_amdgcn_update_dpp(0.0f, x, 0xB1, 0xf, 0xf, false);      // quad_perm: lane ^ 1
        }
        // lane row r = lane / 16 holds fields f, f + 2, f + 4 (f + 4 < its half's end)
        const int r = lane >> 4, f = (r & 1) + (kFields / 2) * (r >> 1);
        const uint32_t slot = __float_as_uint(b.w);
        // every lane has read its rows before any lane overwrites one
        __asm__ volatile("" ::"v"(out[0]), "v"(out[1]), "v"(out[2]), "v"(slot));
        __builtin_amdgcn_wave_barrier();
        if (tj < nb) {
            float* row = reinterpret_cast<float*>(&st.r[0][0]) + 12 * (top - tj) + f;
            row[(lane & 1) ? 2 : 0] = (lane & 1) ? out[1] : out[0];
            if ((lane & 1) == 0 && (kAbs || !(r & 1))) row[4] = out[2];
            if (kAbs ? lane < 16 : f == 0) (kAbs ? st.slot[top - tj] : reinterpret_cast<uint32_t*>(row)[10]) = slot;
        }
        __builtin_amdgcn_wave_barrier();
    };

    // chunk [b_end - 64, b_end) of positions, clipped at lo, walked from the
    // back; lane l of a chunk gathers position b_start + l
    auto chunk_slot = [&](int b_end_) {
        const int b_start_ = max(lo, b_end_ - kChunk);
        return b_end_ > lo ? load_slot(pair_vals, rg.x + (uint32_t)(b_start_ + lane), rg.x + (uint32_t)b_end_) : kNoSlot;
    };
    // adds the reduced rows [r0, r1) of the staged chunk to grad2d, four rows
    // (16 lanes each) at a time
    auto flush = [&](int r0, int r1) {
        const int f = lane & 15;
        if (f < kFields)
            for (int r = r0 + (lane >> 4); r < r1; r += 4) {
                const float* row = reinterpret_cast<const float*>(&st.r[r][0]);
                const uint32_t slot = kAbs ? st.slot[r] : __float_as_uint(row[10]);
                if (row[f] != 0.0f) atomicAdd(&grad2d[(size_t)slot * kG2 + f], row[f]);
            }
        __builtin_amdgcn_wave_barrier();
    };

    // One entry at the lane's pixel, as far as it does not depend on the
    // entries behind it.  An entry the pixel did not composite takes alpha =
    // 0, which leaves T and S unchanged exactly; its dp is left out, not
    // multiplied by 0 (kr is not finite where the gradient of alpha is not).
    struct Step {
        float al, r, kr, gc;
        bool grad, any;
    };
    const float K = gA * (T * Q);      // dL/dalpha_i holds g_alpha T_final / (1 - alpha_i)
    auto step = [&](const float4& a, const float4& b, const float4& c) {
        Step p;
        const Eval e = eval_entry(a, b, pc.fpx, pc.fpy);
        const bool con = __float_as_int(c.w) <= last && e.keep;      // c.w: 1-based position
        p.any = __ballot(con) != 0;
        p.al = con ? e.alpha : 0.0f;
        p.grad = con && e.raw < kAlphaMax;                           // no gradient through the clamp
        const float om = 1.0f - p.al;
        p.r = __builtin_amdgcn_rcpf(om);
        if (kLong) p.r = fmaf(p.r, fmaf(-om, p.r, 1.0f), p.r);
        p.kr = K * p.r;
        p.gc = fmaf(gC0, c.x, fmaf(gC1, c.y, fmaf(gC2, c.z, gD * b.z)));   // g . (colour, depth)
        return p;
    };
    GatherBwd cur = load_entry_bwd(rec, chunk_slot(hi));
    uint32_t s_next = chunk_slot(hi - kChunk);
    int r0 = 0, r1 = 0;      // reduced rows of the staged chunk
    for (int b_end = hi; b_end > lo; b_end -= kChunk) {
        const int b_start = max(lo, b_end - kChunk);
        // Wait for this chunk's records here, then issue the previous
        // chunk's atomics: loads and atomics share one in-order counter, so
        // atomics issued before the wait would be waited for as well.
        __asm__ volatile("" ::"v"(cur.r0.x), "v"(cur.r1.x), "v"(cur.r2.x), "v"(cur.r3.x), "v"(s_next));
        flush(r0, r1);
        const int n = stage_gathered_bwd(cur, b_start + lane + 1, pc, lane, st);
        r0 = r1 = n;
        cur = load_entry_bwd(rec, s_next);
        s_next = chunk_slot(b_end - 2 * kChunk);
        if (n == 0) continue;
        int nb = 0;
        uint64_t ks = 0;
        // entry k - 1 is read from LDS during entry k's update
        Step p = step(st.r[n - 1][0], st.r[n - 1][1], st.r[n - 1][2]);
        const float4* rn = &st.r[n - 1][0];
        float* q = st.q + lane;
        for (int k = n - 1; k >= 0; --k) {
            rn -= k > 0 ? 3 : 0;
            const float4 a = rn[0], b = rn[1], c = rn[2];
            const float Ti = T * p.r;
            const float df = p.gc - S;
            const float dp = p.grad ? fmaf(Ti, df, p.kr) * p.al : 0.0f;       // dL/d power (natural-log units)
            q[0] = dp;
            q[kQW] = p.al * Ti;
            S = fmaf(p.al, df, S);
            T = Ti;
            const bool any = p.any;
            p = step(a, b, c);
            if (any) {
                ks |= (uint64_t)k << (8 * nb);
                q += kQRow;
                if (++nb == kBatch) {
                    reduce(kBatch, ks, r0 - 1);
                    r0 -= kBatch;
                    q = st.q + lane;
                    nb = 0;
                    ks = 0;
                }
            }
        }
        if (nb) {
            reduce(nb, ks, r0 - 1);
            r0 -= nb;
        }
    }
    flush(r0, r1);
}

// Segments per tile in launch order (ceil(L / seg_len) for a list of L > seg_len
// positions, else 1) and the stored states (segments 1 .. n - 1); exclusive
// prefix sums into work_off / state_off.  kSegLenSmall gives way to kSegLen where
// it would store more than kSegStatesSmall states.  When the states would exceed
// `capacity`, every tile keeps a single segment.  A workgroup takes kPlanSpan
// positions, kPlanPer consecutive ones per thread, so that the order is read and
// the offsets are written in whole lines; with several workgroups a first launch
// leaves their sums, which each then adds up itself.  100k tiles: 153 -> 14 us,
// 8160: 17 -> 12 (one workgroup walked the positions, bound by one compute unit's
// range gathers).
constexpr int kPlanThreads = 256, kPlanPer = 8, kPlanSpan = kPlanThreads * kPlanPer;

struct PlanSum {
    uint32_t longest;                    // list
    uint32_t items[2], end_long[2];      // segments, position after the last list with several; of seg_len
};                                       // positions, and of the length that seg_len may give way to

__device__ __forceinline__ uint32_t plan_alternative(uint32_t seg_len) {
    return seg_len == (uint32_t)kSegLenSmall ? (uint32_t)kSegLen : seg_len;
}

__device__ __forceinline__ uint32_t segments_of(uint32_t L, uint32_t seg_len) {
    return L > seg_len ? (L + seg_len - 1) >> __builtin_ctz(seg_len) : 1u;
}

// of positions i0 .. i0 + kPlanPer - 1; L: their lists' lengths
__device__ __forceinline__ PlanSum plan_positions(const uint2* __restrict__ ranges,
                                                  const uint32_t* __restrict__ tile_order, const ViewTable& vt,
                                                  uint32_t seg_len, uint32_t i0, uint32_t L[kPlanPer]) {
    const uint32_t n_tiles = (uint32_t)vt.total_tiles;
    int t[kPlanPer];
#pragma unroll
    for (int u = 0; u < kPlanPer; ++u) t[u] = i0 + u < n_tiles ? order_tile(tile_order, vt, i0 + u) : -1;
    uint2 r[kPlanPer];
#pragma unroll
    for (int u = 0; u < kPlanPer; ++u) r[u] = t[u] >= 0 ? ranges[t[u]] : make_uint2(0u, 0u);
    PlanSum s{0u, {0u, 0u}, {0u, 0u}};
#pragma unroll
    for (int u = 0; u < kPlanPer; ++u) {
        L[u] = r[u].y - r[u].x;
        s.longest = max(s.longest, L[u]);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint32_t c = t[u] < 0 ? 0u : segments_of(L[u], k ? plan_alternative(seg_len) : seg_len);
            if (c > 1u) s.end_long[k] = i0 + u + 1;
            s.items[k] += c;
        }
    }
    return s;
}

// of two parts of the positions
__device__ __forceinline__ PlanSum plan_join(PlanSum a, const PlanSum& b) {
    a.longest = max(a.longest, b.longest);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        a.items[k] += b.items[k];
        a.end_long[k] = max(a.end_long[k], b.end_long[k]);
    }
    return a;
}

// over the workgroup, in every thread (s: one a wave)
__device__ __forceinline__ PlanSum plan_reduce(PlanSum v, PlanSum* s) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        PlanSum y;
        y.longest = (uint32_t)__shfl_xor((int)v.longest, off, 64);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            y.items[k] = (uint32_t)__shfl_xor((int)v.items[k], off, 64);
            y.end_long[k] = (uint32_t)__shfl_xor((int)v.end_long[k], off, 64);
        }
        v = plan_join(v, y);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    v = s[0];
#pragma unroll
    for (int w = 1; w < kPlanThreads / 64; ++w) v = plan_join(v, s[w]);
    return v;
}

__global__ __launch_bounds__(kPlanThreads) void k_seg_sums(const uint2* __restrict__ ranges,
                                                           const uint32_t* __restrict__ tile_order, ViewTable vt,
                                                           uint32_t seg_len, PlanSum* __restrict__ sums) {
    __shared__ PlanSum s_red[kPlanThreads / 64];
    uint32_t L[kPlanPer];
    const PlanSum v = plan_reduce(plan_positions(ranges, tile_order, vt, seg_len,
                                                 blockIdx.x * kPlanSpan + threadIdx.x * kPlanPer, L), s_red);
    if (threadIdx.x == 0) sums[blockIdx.x] = v;
}

__global__ __launch_bounds__(kPlanThreads) void k_seg_plan(const uint2* __restrict__ ranges,
                                                           const uint32_t* __restrict__ tile_order, ViewTable vt,
                                                           uint32_t seg_len, uint32_t capacity,
                                                           const PlanSum* __restrict__ sums,
                                                           uint32_t* __restrict__ work_off,
                                                           uint32_t* __restrict__ state_off, uint32_t* __restrict__ info) {
    __shared__ PlanSum s_red[kPlanThreads / 64];
    __shared__ uint32_t s_wave[kPlanThreads / 64];
    const uint32_t n_tiles = (uint32_t)vt.total_tiles;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t i0 = blockIdx.x * kPlanSpan + threadIdx.x * kPlanPer;
    uint32_t L[kPlanPer];
    const PlanSum mine = plan_positions(ranges, tile_order, vt, seg_len, i0, L);
    // segments of the earlier workgroups, and of all
    PlanSum all = mine, early{0u, {0u, 0u}, {0u, 0u}};
    if (gridDim.x > 1) {
        all = early;
        for (uint32_t b = threadIdx.x; b < gridDim.x; b += kPlanThreads) {
            const PlanSum x = sums[b];
            if (b < blockIdx.x) early = plan_join(early, x);
            all = plan_join(all, x);
        }
        early = plan_reduce(early, s_red);
    }
    all = plan_reduce(all, s_red);
    const bool other = all.items[0] - n_tiles > (uint32_t)kSegStatesSmall;
    const uint32_t len = other ? plan_alternative(seg_len) : seg_len;
    const uint32_t items = other ? all.items[1] : all.items[0];
    const uint32_t end_long = other ? all.end_long[1] : all.end_long[0];
    const uint32_t here = other ? mine.items[1] : mine.items[0];
    // exclusive scan over the workgroup's threads
    uint32_t incl = here;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint32_t w = (other ? early.items[1] : early.items[0]) + incl - here;
    for (int k = 0; k < wave; ++k) w += s_wave[k];
    const uint32_t need = items - n_tiles;
    const bool on = need <= capacity;      // do the states fit?
#pragma unroll
    for (int u = 0; u < kPlanPer; ++u) {
        if (i0 + u >= n_tiles) break;
        work_off[i0 + u] = on ? w : i0 + u;
        state_off[i0 + u] = on ? w - (i0 + u) : 0u;
        w += segments_of(L[u], len);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        work_off[n_tiles] = on ? items : n_tiles;
        state_off[n_tiles] = on ? need : 0u;
        info[kPlanLong] = on ? end_long : 0u;
        // lists up to kHeadLen are composited by the head alone when none is
        // longer: the later passes cost more than a head that long
        info[kPlanHead] = segments_of(all.longest, len) * len > (uint32_t)kHeadLen ? 2u : (uint32_t)kHeadLen / len;
        info[kPlanLen] = len;
    }
}

// State of one stored segment (tile at launch position i, segment j >= 1):
// per pixel, front to back over the segment's composited entries (position
// <= last and not skipped), T_seg = prod (1 - alpha) and the colour and
// depth sums with T restarted at 1: C_seg = sum c alpha T_local.  The
// alpha values are the forward's and the backward's bit for bit.
__global__ __launch_bounds__(256) void k_seg_prepass(const float4* __restrict__ rec,
                                                     const uint32_t* __restrict__ pair_vals,
                                                     const uint2* __restrict__ ranges,
                                                     const uint32_t* __restrict__ tile_order, ViewTable vt,
                                                     const int32_t* __restrict__ last_in, SegPlan plan) {
    __shared__ WaveStage stage[kWaves];
    const uint32_t b = blockIdx.x;
    if (b >= plan.state_off[plan.n_tiles]) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t i = last_le_wave(plan.state_off, plan.info[kPlanLong], b, lane);
    const int j = (int)(b - plan.state_off[i]) + 1;
    const int tile = order_tile(tile_order, vt, i);
    const PixelCoords pc = pixel_coords(vt, tile, wave, lane);
    WaveStage& st = stage[wave];
    const uint2 rg = ranges[tile];
    const int last = pc.inside ? last_in[pc.pix] : 0;
    int maxlast = last;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) maxlast = max(maxlast, __shfl_xor(maxlast, off, 64));
    const int seg_len = (int)plan.info[kPlanLen], lo = j * seg_len, hi = min(lo + seg_len, maxlast);
    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, D = 0.0f;
    for (int b0 = lo; b0 < hi; b0 += kChunk) {
        const Gather e = load_entry(rec, load_slot(pair_vals, rg.x + (uint32_t)(b0 + lane), rg.x + (uint32_t)hi));
        const int n = stage_gathered(e, b0 + lane + 1, pc, lane, st);
        for (int k = 0; k < n; ++k) {
            const float4 a = st.g[k], bb = st.b[k], c = st.c[k];
            const Eval ev = eval_entry(a, bb, pc.fpx, pc.fpy);
            const bool con = __float_as_int(c.w) <= last && ev.keep;
            const float w = con ? ev.alpha * T : 0.0f;
            c0 = fmaf(c.x, w, c0);
            c1 = fmaf(c.y, w, c1);
            c2 = fmaf(c.z, w, c2);
            D = fmaf(bb.z, w, D);
            T = con ? T * (1.0f - ev.alpha) : T;
        }
        __builtin_amdgcn_wave_barrier();
    }
    float* out = plan.state + (size_t)b * kSegFields * 256;
    const int px = pc.ly * kTile + pc.lx;
    out[0 * 256 + px] = T;
    out[1 * 256 + px] = c0;
    out[2 * 256 + px] = c1;
    out[3 * 256 + px] = c2;
    out[4 * 256 + px] = D;
}

// 2D-gradient rows of the slots that some tile lists (tiles > 0): the only
// rows the compositing backward accumulates into and the only ones read
__global__ __launch_bounds__(256) void k_zero_seen_rows(const uint32_t* __restrict__ tiles, float4* __restrict__ grad2d,
                                                        int64_t n_slots) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_slots || tiles[i] == 0) return;
    const float4 z = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    grad2d[3 * i + 0] = z;
    grad2d[3 * i + 1] = z;
    grad2d[3 * i + 2] = z;
}

}  // namespace

hipError_t launch_render_fwd(const Projected& proj, const uint32_t* pair_vals, const uint2* ranges,
                             const ViewTable& vt, const OptK& opt, float* rgb, float* depth, float* alpha,
                             float* T_final, int32_t* last, hipStream_t s, int persistent_ctas, uint32_t* work,
                             const SegPlan* plan) {
    if (vt.total_tiles <= 0) return hipSuccess;
    const hipEvent_t timed_ = timer_begin(GS_KERNEL_RENDER_FWD, s);
    if (persistent_ctas > 0 && work) {
        hipError_t e = fill_u32(work, 0u, 1, s);
        if (e != hipSuccess) return e;
        const int grid = persistent_ctas < vt.total_tiles ? persistent_ctas : vt.total_tiles;
        hipLaunchKernelGGL(k_render_fwd_persistent, dim3(grid), dim3(256), 0, s, proj.rec, pair_vals, ranges,
                           proj.tile_order, vt, opt, rgb, depth, alpha, T_final, last, work);
    } else {
        const SegPlan none{nullptr, nullptr, nullptr, (uint32_t)vt.total_tiles, nullptr, 0u, nullptr, (uint32_t)kSegLen};
        hipLaunchKernelGGL(k_render_fwd, dim3(vt.total_tiles), dim3(256), 0, s, proj.rec, pair_vals, ranges,
                           proj.tile_order, vt, opt, rgb, depth, alpha, T_final, last, plan ? *plan : none);
        if (plan && plan->capacity) {
            // the later segments of the planned lists, the fold, and the
            // re-walk of the segments pixels stop in
            hipLaunchKernelGGL(k_fwd_segments, dim3(plan->capacity), dim3(256), 0, s, proj.rec, pair_vals, ranges,
                               proj.tile_order, vt, *plan);
            hipLaunchKernelGGL(k_fwd_combine, dim3(vt.total_tiles), dim3(256), 0, s, proj.tile_order, vt, opt, *plan,
                               rgb, depth, alpha, T_final, last);
            hipLaunchKernelGGL(k_fwd_fix, dim3(plan->capacity), dim3(256), 0, s, proj.rec, pair_vals, ranges,
                               proj.tile_order, vt, opt, *plan, rgb, depth, alpha, T_final, last);
        }
    }
    timer_end(timed_, s);
    return hipGetLastError();
}

hipError_t launch_render_count(const Projected& proj, const uint32_t* pair_vals, const uint2* ranges,
                               const ViewTable& vt, int32_t* n_eval, hipStream_t s) {
    if (vt.total_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_render_count, dim3(vt.total_tiles), dim3(256), 0, s, proj.rec, pair_vals, ranges,
                       proj.tile_order, vt, n_eval);
    return hipGetLastError();
}

hipError_t launch_seg_plan(const Projected& proj, const uint2* ranges, const ViewTable& vt, uint32_t capacity,
                           const SegPlan& plan, hipStream_t s) {
    const unsigned blocks = (unsigned)((vt.total_tiles + kPlanSpan - 1) / kPlanSpan);
    // the sums lie where the forward's stop_seg will (1 KB a tile)
    PlanSum* sums = reinterpret_cast<PlanSum*>(plan.stop_seg);
    if (blocks > 1)
        hipLaunchKernelGGL(k_seg_sums, dim3(blocks), dim3(kPlanThreads), 0, s, ranges, proj.tile_order, vt, plan.seg_len,
                           sums);
    hipLaunchKernelGGL(k_seg_plan, dim3(blocks ? blocks : 1u), dim3(kPlanThreads), 0, s, ranges, proj.tile_order, vt,
                       plan.seg_len, capacity, sums, plan.work_off, plan.state_off, plan.info);
    return hipGetLastError();
}

hipError_t launch_seg_prepare(const Projected& proj, const uint32_t* pair_vals, const uint2* ranges,
                              const ViewTable& vt, const int32_t* last, uint32_t capacity, const SegPlan& plan,
                              hipStream_t s) {
    hipError_t e = launch_seg_plan(proj, ranges, vt, capacity, plan, s);
    if (e != hipSuccess) return e;
    if (capacity)
        hipLaunchKernelGGL(k_seg_prepass, dim3(capacity), dim3(256), 0, s, proj.rec, pair_vals, ranges, proj.tile_order,
                           vt, last, plan);
    return hipGetLastError();
}

hipError_t launch_render_bwd(const Projected& proj, const uint32_t* pair_vals, const uint2* ranges,
                             const ViewTable& vt, const OptK& opt, const float* T_final, const int32_t* last,
                             const float* d_rgb, const float* d_depth, const float* d_alpha, float* grad2d,
                             const SegPlan& plan, uint32_t capacity, bool abs_sums, hipStream_t s) {
    // with a plan, blocks beyond the planned work items exit at once
    const unsigned blocks = wave_grid((unsigned)vt.total_tiles + (plan.work_off ? capacity : 0u));
    const hipEvent_t timed_ = timer_begin(GS_KERNEL_RENDER_BWD, s);
    const bool longer = plan.work_off && plan.seg_len > (uint32_t)kSegLen;
    const auto kernel = abs_sums ? (longer ? k_render_bwd<true, true> : k_render_bwd<true, false>)
                                 : (longer ? k_render_bwd<false, true> : k_render_bwd<false, false>);
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(64), 0, s, proj.rec, pair_vals, ranges, proj.tile_order, vt, opt, T_final,
                       last, d_rgb, d_depth, d_alpha, grad2d, plan);
    timer_end(timed_, s);
    return hipGetLastError();
}

hipError_t zero_seen_grad2d(const uint32_t* tiles, float* grad2d, int64_t n_slots, hipStream_t s) {
    const unsigned blocks = (unsigned)((n_slots + 255) / 256);
    hipLaunchKernelGGL(k_zero_seen_rows, dim3(blocks), dim3(256), 0, s, tiles, reinterpret_cast<float4*>(grad2d),
                       n_slots);
    return hipGetLastError();
}

}  // namespace gs
