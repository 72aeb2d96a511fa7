// Internal declarations of the MI355X renderer: workspace layout, the BVH
// descriptor, record layouts and small device helpers shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "raysplats.h"

namespace rs {

constexpr uint64_t kMagic = 0x5253425648495031ull;  // "RSBVHIP1"
constexpr int kWave = 64;
constexpr int kMaxSets = 2 * RS_MAX_BOUNCES + 1;  // ray sets one render launch can carry (mesh path + shadow rays)
constexpr int kXcdQueues = 8;  // persistent packet queues (one per XCD of MI355X)
constexpr int kStripTiles = 16;  // persistent packet order: strips 16 tiles wide

// log2 of the packet tile width of a launch (tile_width 0 = 8x8 tiles)
inline int tile_shift_of(const rs_params *p)
{
    switch (p ? p->tile_width : 0) {
    case 4: return 2;
    case 16: return 4;
    case 32: return 5;
    default: return 3;
    }
}
// log2 of the rays per packet of a launch over `sets` ray sets. A launch needs some thousands of packets to
// fill the chip, and the rays of a small image lie far apart, so a 64-ray packet of one spans a wide
// bundle: launches of few rays, and those over small views of large scenes, trace 16-ray packets.
// Forward and adjoint, 16-ray against 64-ray packets: 3000 Gaussians, 77k rays 0.30 and 0.33 ms, 128k rays
// 0.40 and 0.33; 300k, 480x320 2.6 and 4.1; 500k, 640x480 4.9 and 4.2; 1M, 480x320 7.4 and 13.6, 640x480 8.1
// and 8.1; 260k, three views of 406x228 and four of 203x85 6.3 and 12.9. The paper variant keeps 64: its
// pool bound counts on 64-ray rows. So does brute force, whose packets each test every Gaussian (20k, 98304 rays:
// 12.9 ms, 22.2 in 16-ray packets).
constexpr int64_t kSmallLaunchRays = 98304, kMidLaunchRays = 524288, kSmallViewRays = 196608;
inline int packet_shift(const rs_rays *rays, int64_t sets, const rs_params *p, int64_t n_gauss)
{
    if (p && (p->flags & (RS_PAPER_GRADIENT | RS_BRUTE_FORCE))) return 6;
    const int64_t n = rays->n * sets, per_view = rays->n / (rays->n_views > 0 ? rays->n_views : 1);
    const bool small_views = n <= kMidLaunchRays && per_view <= kSmallViewRays && n_gauss >= per_view;
    return n <= kSmallLaunchRays || small_views ? 4 : 6;
}
// The same for a pass that neither writes nor reads stored lists (whose rows name lanes of the
// packets that wrote them): where the Gaussians far outnumber the rays, even 16-ray packets are wide,
// and 4-ray ones are faster. Forward with 4-ray and 16-ray packets, by Gaussians per ray: 17 (1M, 320x180) 2.2 and 5.7 ms;
// 5.2 (100k, 160x120) 0.99 and 1.48; 5.2 (300k, 320x180) 1.70 and 1.33; 4.1 (200k, 256x192) 0.83 and 0.95; 3.5 (200k,
// 320x180) 0.71 and 1.00; 3.3 (100k, 200x150) 1.89 and 1.17; 2.0 (100k, 256x192) 1.76 and 0.96; 1.1 (100k, 360x260) 2.03
// and 1.07. Random pixels are faster in 4-ray packets on either side (4.6: 10.0 and 13.7; 3.1: 5.2 and 7.8).
inline int packet_shift_no_lists(const rs_rays *rays, int64_t sets, const rs_params *p, int64_t n_gauss)
{
    const int ps = packet_shift(rays, sets, p, n_gauss);
    return ps == 4 && n_gauss >= 4 * rays->n * sets ? 2 : ps;
}
// Scenes of up to this many Gaussians are walked where a launch has packets enough to fill the chip: a frontier
// has fixed costs (1000 Gaussians, 588x587: 100 us walked, 115 in windows; 3000: 248 and 232).
constexpr int64_t kFrontFew = 2048;
// Whether a forward pass takes the frontier kernel. It keeps no stack: a call that bounds the stack takes the walk. So
// does the paper variant (its pool bound, see k_render), and so do the sets of paths of several bounces: refracted
// rays of a packet go all ways (150k Gaussians, 640x361, three bounces: 7.7 ms walked, 9.2 to 22 otherwise).
inline bool front_route(const rs_rays *rays, int sets, const rs_params *p, int64_t n_gauss, bool lists)
{
    return !(p->flags & RS_BRUTE_FORCE) && !((p->flags & RS_PAPER_GRADIENT) && lists) && p->stack_depth == 0 && sets <= 3 &&
           (n_gauss > kFrontFew || packet_shift(rays, sets, p, n_gauss) < 6);
}
// The hits that a frontier's buffer holds for a kbuf.
inline int front_keys(int kbuf) { return kbuf == 0 ? 24 : kbuf <= 16 ? 16 : kbuf <= 24 ? 24 : 32; }
constexpr int kSortBlock = 256;
constexpr int kSortItems = 8;  // keys per thread per sort tile
constexpr int kSortTile = kSortBlock * kSortItems;

// PLOC build: neighbourhood radius, clusters per workgroup of the grid-wide
// iterations (small chunks keep every workgroup short once few clusters are
// left), the finish kernel's LDS capacity, workgroup sizes.
constexpr int kPlocR = 8;
constexpr int kPlocChunk = 512;
constexpr int kPlocThreads = 256;
constexpr int kPlocLocal = 4096;
constexpr int kPlocFinishThreads = 1024;
constexpr int kPlocMaxIters = 512;  // size of the per-iteration control array

// ceil(log2(ceil(n / kPlocLocal))) for n > kPlocLocal, else 0
inline int ploc_halvings(int64_t n)
{
    if (n <= kPlocLocal) return 0;
    const int64_t c = (n + kPlocLocal - 1) / kPlocLocal;
    int l = 0;
    while ((int64_t(1) << l) < c) ++l;
    return l;
}
// Grid-wide iterations launched for n clusters (the clustering removes about
// a tenth of the clusters per iteration; whatever is left above kPlocLocal
// afterwards is finished from global memory).
inline int ploc_global_iters(int64_t n) { return 7 * ploc_halvings(n); }
// Iteration from which clusters are paired by position instead of by
// distance, so every build ends after a bounded number of iterations.
inline int ploc_cap(int64_t n) { return 256 + 10 * ploc_halvings(n); }

// Device status bits (sticky, OR-ed by kernels).
constexpr int kStatusStack = 1;
constexpr int kStatusNonfinite = 2;
constexpr int kStatusListPool = 4;  // RS_PAPER_GRADIENT: the stored-list pool ran out

// Gaussian record, one per sorted position (64 bytes, four float4):
//   r0 = (RT00, RT01, RT02, RT10), r1 = (RT11, RT12, RT20, RT21),
//   r2 = (RT22, 1/sx, 1/sy, 1/sz), r3 = (mx, my, mz, opacity)
// RT = R^T, R the rotation of the normalised quaternion.
// BVH node, one per internal node (64 bytes, four float4):
//   n0 = (L.lo.x, L.lo.y, L.lo.z, L.hi.x), n1 = (L.hi.y, L.hi.z, R.lo.x, R.lo.y),
//   n2 = (R.lo.z, R.hi.x, R.hi.y, R.hi.z), n3 = (left ref, right ref, -, -) as int bits
// A child ref >= 0 names an internal node; ref < 0 names leaf ~ref.

// Header block at the start of the workspace (256 bytes).
struct WsHeader {
    int32_t status;
    uint32_t queue;        // persistent packet counter
    uint32_t bounds[6];    // ordered-uint min xyz, max xyz of the means
    float root_box[6];
    uint64_t counters[16];  // instrumentation (RS_COUNTERS)
    uint32_t xq[8];         // persistent packet counters, one per XCD chunk
    uint32_t pad[10];
};
static_assert(sizeof(WsHeader) == 256, "header size");

struct Layout {
    size_t header, records, nodes, gidx, inv, codes, leaf_boxes, parent, visit, ibox, keys_alt, vals_alt, hist, totals, gacc;
    size_t ploc_box, ploc_ref, ploc_pm, ploc_blk, ploc_ctrl, total;
    int64_t n, n_int, sort_blocks, ploc_chunks;
};

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

inline Layout make_layout(int64_t n)
{
    Layout L{};
    L.n = n;
    L.n_int = n > 1 ? n - 1 : 0;
    int64_t nn = n > 0 ? n : 1;
    int64_t ni = L.n_int > 0 ? L.n_int : 1;
    L.sort_blocks = (nn + kSortTile - 1) / kSortTile;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align256(off + bytes);
        return o;
    };
    L.header = take(sizeof(WsHeader));
    L.records = take(size_t(nn) * 64);
    L.nodes = take(size_t(ni) * 64);
    L.gidx = take(size_t(nn) * 4);
    L.inv = take(size_t(nn) * 4);
    L.codes = take(size_t(nn) * 4);
    L.leaf_boxes = take(size_t(nn) * 24);
    L.parent = take(size_t(2 * nn) * 4);
    L.visit = take(size_t(ni) * 4);
    L.ibox = take(size_t(ni) * 24);
    L.keys_alt = take(size_t(nn) * 4);
    L.vals_alt = take(size_t(nn) * 4);
    L.hist = take(size_t(256) * L.sort_blocks * 4);
    L.totals = take(size_t(512) * 4);
    L.gacc = take(size_t(nn) * 64);
    // PLOC clusters: two buffers of boxes (6 float arrays of n each) and refs,
    // the merge code per position, per-chunk counts, per-iteration control
    L.ploc_chunks = (nn + kPlocChunk - 1) / kPlocChunk;
    L.ploc_box = take(size_t(nn) * 48);
    L.ploc_ref = take(size_t(nn) * 8);
    L.ploc_pm = take(size_t(nn) * 4);
    L.ploc_blk = take(size_t(L.ploc_chunks) * 8);
    L.ploc_ctrl = take(size_t(kPlocMaxIters) * 16);
    L.total = off;
    return L;
}

// Descriptor stored in rs_bvh.opaque.
struct BvhDesc {
    uint64_t magic;
    int64_t n;
    float Q;
    int32_t root;       // root ref (0: internal node 0; ~0: single leaf; unused when n == 0)
    char *ws;
    uint64_t ws_bytes;
    int32_t kind;       // kKindGaussians or kKindMesh
    int32_t pad0;
    uint64_t pad[9];
};
constexpr int32_t kKindGaussians = 1;
constexpr int32_t kKindMesh = 2;
static_assert(sizeof(BvhDesc) <= sizeof(rs_bvh), "descriptor size");

// ---------------------------------------------------------------- helpers

// Wave-wide vote as a plain 64-bit lane mask (no int materialisation of the
// predicate, unlike the generic ballot).
__device__ inline uint64_t wave_ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

__device__ inline uint32_t float_to_ordered(float f)
{
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ inline float ordered_to_float(uint32_t u)
{
    uint32_t b = (u & 0x80000000u) ? (u & 0x7fffffffu) : ~u;
    return __uint_as_float(b);
}

// Ray state of one ray set (caller-owned), 256-byte aligned sections:
//   fin[n]   float4: final colour (composite + T bg) and final transmittance T
//   last[n]  uint4: the last composited hit's key (low word: Gaussian index,
//            high word: float bits of t1 + bias; both 0 when nothing was
//            composited), then T just before the hit that took T below the
//            smallest normal float (to 0 when alpha = 1) and the number of
//            composited hits after that one (0xffffffff when T stayed normal).
//            The adjoint walks the hits back to front from that key and
//            recovers T_k = T_{k+1} / (1 - alpha_k) from the final T; the saved
//            T restarts the recursion where it would divide 0 by 0 or lose its
//            digits in the subnormals.
//   list[n]  int4 (only with stored hit lists): composited hits, how many of
//            them the pool holds, the ray's packet's last pool chunk and the
//            packet's stored row count.
struct SetState {
    float4 *fin;
    uint4 *last;
    int4 *list;
};

// Stored hit lists: one pool shared by every packet of a launch. A packet's
// wavefront appends, per compositing step, the entries of the lanes that
// consumed a hit at that step, in lane order (the Gaussian index it composited,
// or the index | kListSecond for a hit it only collected in the paper variant's
// second phase). A row is one step of a 64-ray packet, or up to four of a 16-ray one,
// and ends with 64 mask bits as two words: the lanes of its step, or 16 bits a step. With a row per step a
// 16-ray packet's masks took a quarter of its slots, and pools that suffice for 64-ray packets ran out
// (list adjoint of 96x96 rays with mirrors, 500,000 Gaussians, 64 slots a ray: 6.35 -> 0.75 ms; where the pool
// sufficed, 16-ray packets' adjoint is 4 % faster, 0.347 -> 0.333 ms at 251x187 over 20,000).
// Rows are packed into chunks of 4-byte slots (8 per ray of a packet; a row never straddles two
// chunks), linked backwards per packet; fill[c] is the number of slots chunk c
// holds. The pool header holds the chunk counter (64-bit) and a flag set when a
// packet found the pool exhausted (its later rows are not stored).
constexpr int kChunkSlots = 512;  // the unit in which pools are sized, and a chunk of 64-ray packets
constexpr int kRowSteps = 4;      // steps in a row of a 16-ray packet
inline int chunk_slots_of(int pkt_shift) { return kChunkSlots >> (6 - pkt_shift); }
constexpr uint32_t kListIdle = 0xffffffffu;
constexpr uint32_t kListSecond = 0x80000000u;
struct ListPool {
    unsigned long long *hdr;  // [0] chunks taken, [1] exhausted flag; its upper half: log2 of the rays per packet
    int32_t *prev;            // [chunks] previous chunk of the same packet (-1: first)
    int32_t *fill;            // [chunks] slots used
    uint32_t *slots;          // [chunks][chunk_slots]
    int64_t chunks;
    int32_t chunk_slots;  // kChunkSlots: 64-ray packets, a row a step
};
inline int64_t list_chunks(int64_t slots_wanted)
{
    return (slots_wanted + kChunkSlots - 1) / kChunkSlots;
}
// bytes of a pool of `chunks` chunks (header, links, fills, slots), 256-byte aligned
inline size_t list_pool_bytes(int64_t chunks)
{
    if (chunks <= 0) return 0;
    return 256 + 2 * align256(size_t(chunks) * 4) + size_t(chunks) * kChunkSlots * 4;
}
// Where a pool lies: the bytes of `units` chunks of kChunkSlots slots (list_pool_bytes). The launch carves them,
// since the packet size depends on the scene too.
struct ListRoom {
    char *base;
    int64_t units;
};
// The pool in the bytes of `units` chunks of kChunkSlots slots. Smaller chunks have more links and
// fills: as many chunks as then fit.
inline ListPool list_pool_at(const ListRoom &at, int chunk_slots)
{
    char *base = at.base;
    const int64_t units = at.units;
    ListPool P{};
    if (!base || units <= 0) return P;
    const size_t room = list_pool_bytes(units) - 256;
    int64_t chunks = units;
    if (chunk_slots != kChunkSlots) {
        chunks = int64_t(room / (size_t(chunk_slots) * 4 + 8));
        while (2 * align256(size_t(chunks) * 4) + size_t(chunks) * chunk_slots * 4 > room) --chunks;
    }
    P.hdr = reinterpret_cast<unsigned long long *>(base);
    P.prev = reinterpret_cast<int32_t *>(base + 256);
    P.fill = reinterpret_cast<int32_t *>(base + 256 + align256(size_t(chunks) * 4));
    P.slots = reinterpret_cast<uint32_t *>(base + 256 + 2 * align256(size_t(chunks) * 4));
    P.chunks = chunks;
    P.chunk_slots = chunk_slots;
    return P;
}

// Host description of one ray set of a render launch.
struct SetDesc {
    const rs_rays *rays;
    float *out_rgb;   // forward output (may be null in the adjoint)
    SetState state;   // fin may be null: no state written (forward without adjoint)
    const float *grad;
    float bg[3];
    int32_t zero_colour;
};

// Layout of the caller's ray state for n rays and hit-list capacity C
// (pool of C slots per ray on average).
struct StateLayout {
    size_t fin, last, list, pool, total;
    int64_t chunks;
};
inline StateLayout state_layout(int64_t n, int32_t cap)
{
    StateLayout L{0, 0, 0, 0, 0, 0};
    const size_t nn = size_t(n > 0 ? n : 0);
    L.fin = 0;
    L.last = align256(nn * 16);
    L.total = L.last + nn * 16;
    if (cap <= 0 || nn == 0) return L;
    L.list = align256(L.total);
    L.pool = align256(L.list + nn * 16);
    L.chunks = list_chunks(int64_t(nn) * cap);
    L.total = L.pool + list_pool_bytes(L.chunks);
    return L;
}
inline SetState state_at(void *base, int64_t n, int32_t cap)
{
    SetState S{nullptr, nullptr, nullptr};
    if (!base || n <= 0) return S;
    const StateLayout L = state_layout(n, cap);
    char *b = static_cast<char *>(base);
    S.fin = reinterpret_cast<float4 *>(b + L.fin);
    S.last = reinterpret_cast<uint4 *>(b + L.last);
    if (L.chunks > 0) S.list = reinterpret_cast<int4 *>(b + L.list);
    return S;
}

// What a render launch does.
enum class Pass { Forward, AdjointList, AdjointTraverse };

int launch_build(const rs_gaussians *g, float Q, bool lbvh, char *ws, hipStream_t st);
int launch_sets(const BvhDesc &D, const rs_gaussians *g, const rs_params *p, int nsets, const SetDesc *sets,
                const ListRoom &room, Pass pass, hipStream_t st);
// zero a pool's header (before a forward that stores lists)
void reset_pool(const ListPool &pool, int pkt_shift, hipStream_t st);
int launch_render(const BvhDesc &D, const rs_gaussians *g, const rs_rays *rays, const rs_params *p, float *out_rgb,
                  void *state, const float *grad, const rs_grads *grads, hipStream_t st);
void zero_gacc(const BvhDesc &D, hipStream_t st);
int launch_build_mesh(const rs_mesh *m, char *ws, hipStream_t st);
int launch_trace_mesh(const BvhDesc &M, const rs_rays *rays, const float *t_limit, int any_hit, int tile_shift, float *t_hit,
                      int32_t *tri, hipStream_t st);
size_t mesh_frame_bytes(int64_t n, int32_t cap, int bounces);
int mesh_frame_set(char *frame, int64_t n, int32_t cap, int bounces, int set, SetState *st, ListRoom *room);
size_t loss_workspace_bytes(int32_t w, int32_t h);
int launch_loss(const float *img, const float *tgt, int32_t w, int32_t h, const rs_loss_params *lp, float *loss,
                float *grad, void *ws, hipStream_t st);
size_t loss_scratch_bytes();
int loss_scratch(void **out);
int launch_mesh_fwd(const BvhDesc &G, const BvhDesc &M, const rs_gaussians *g, const rs_shading *sh,
                    const rs_rays *rays, const rs_params *p, float *out_rgb, void *frame, hipStream_t st);
int launch_mesh_bwd(const BvhDesc &G, const rs_gaussians *g, const rs_shading *sh, const rs_rays *rays, const rs_params *p,
                    const float *grad, void *frame, const rs_grads *grads, hipStream_t st);
void scatter_gacc(const BvhDesc &D, const float *quat, const rs_grads *grads, hipStream_t st);

}  // namespace rs
