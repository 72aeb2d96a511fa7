// Ray-packet traversal, ellipsoid intersection, depth-ordered compositing and
// its adjoint, for gfx950 (wave64).
//
// One wavefront traces one packet of 64 rays (an 8x8 pixel tile; 16 or 4 rays in small launches).
// Each lane keeps its nearest not-yet-composited hits, ordered by the key (t1, Gaussian index), in
// registers, and composites them front to back (Eq. 3) with the K_max and eps1 stops (Sec. 3, "Color
// Aggregation"). There are two ways to find them, with the same result bit for bit:
//
// The frontier kernel (k_render_front, most forward calls) lets the lanes test 64 nodes, then 64
// leaves, at a time against the bundle of the packet's rays, from near to far, and tests the
// leaves that survive ray by ray; hits in front of all open work are composited at once.
//
// The walk (k_render, and the frontier kernel's fallback): the whole wave walks the BVH depth
// first; node and Gaussian records are fetched once per wave (uniform addresses, scalar loads) and
// every lane tests them against its own ray; a child is entered when any lane's ray overlaps it
// (ballot). The traversal stack is wave-uniform and lives in one VGPR (entry k in lane k). A round
// collects the K smallest keys above the previous round's last key (nodes are culled against
// [last t, K-th t]), then composites them. Rounds repeat until every lane has stopped or run out of hits.
//
// The adjoint (App. A.3-A.6) walks each ray's composited hits back to front,
// either from the forward's stored lists or by traversing the BVH again in
// rounds that collect the K largest keys below the previous round's first
// one. The colour seen behind hit k, S_{k+1}, is built back to front
// (S <- alpha c + (1 - alpha) S from the background), so dL/dalpha_k =
// T_k <g, c_k - S_{k+1}> needs no division by 1 - alpha_k. T_k comes from the
// final T as T_{k+1} / (1 - alpha_k) (a relative error of about 2 ulp per
// hit), restarted from the T the forward saved where T left the normal floats
// (reached 0 when alpha = 1, or underflowed). The
// gradients of alpha with respect to the Gaussian parameters follow App. A.6
// in a cancellation-free form (see grad_hit). Per-Gaussian gradient
// contributions of a wave are summed across lanes before one set of float32
// atomics per Gaussian.
#include <math.h>

#include "rs_device.h"

#pragma clang fp contract(on)

namespace rs {

struct RenderParams {
    int64_t n_packets;         // all sets
    int64_t packets_per_set;   // every set has the same ray layout (views / packets)
    int64_t n_rays;            // rays per set
    int64_t n_gauss;
    int32_t root;
    int32_t stack_depth;
    float Q, eps1, t_min;
    int32_t max_hits;
    uint32_t flags;
    int32_t persistent;
    int32_t brute;
    int32_t front;         // forward: the frontier kernel (else the depth-first walk)
    int32_t count;
    int32_t n_views;
    int32_t tile_shift, pkt_shift;
    int32_t strip_tiles;   // persistent: tile strip width of the packet order (0 = row-major)
    int32_t lists;         // stored hit lists: the forward appends rows, the adjoint replays them
    int32_t overflow_only; // traversal adjoint next to stored lists: only rays whose list is incomplete
    int32_t paper;         // RS_PAPER_GRADIENT: second phase after an eps1 stop
    float eps2;
    int64_t chunk;         // persistent: packets per XCD queue
    ViewEntry views[RS_MAX_VIEWS];
};

// ------------------------------------------------------------ intersection

// Ray / confidence-ellipsoid test (Sec. 3, Prop. 1, Prop. 2) for the record
// r0..r3 (R^T, 1/s, mean, opacity). With x = o - m, the whitened ray is
// o' = D R^T x, d' = D R^T d (D = diag(1/s)); its squared distance to the
// origin is h^2 = |o' x d'|^2 / |d'|^2 and o' x d' = cof(D) R^T (x cross d)
// with cof(D) = (D1 D2, D0 D2, D0 D1): every term is a sum of squares, so flat
// Gaussians (one scale -> 0) lose no precision to cancellation. The nearer
// root is t1 = -b/a - sqrt((Q - h^2)/a) for b = <o',d'> >= 0 and the Viete
// form (|o'|^2 - Q) / (a t*) otherwise (Prop. 1, App. A.1).
// Intermediates of the test that the adjoint of a hit reuses (the body-frame
// offset y = R^T (o - m) and direction e = R^T d, the scaled cross product u,
// b = <o',d'>, 1/a).
struct HitGeom {
    float y0, y1, y2, e0, e1, e2, u0, u1, u2, b, ia;
};

// The test in two parts, so a wave can skip the second when no lane's ray meets the ellipsoid.
// First part: the whitened geometry and h^2.
__device__ inline float ellipsoid_h2(const Ray &ray, const float4 r0, const float4 r1, const float4 r2, const float4 r3,
                                     HitGeom &G)
{
    const float xx = ray.ox - r3.x, xy = ray.oy - r3.y, xz = ray.oz - r3.z;
    // rows of R^T
    const float a00 = r0.x, a01 = r0.y, a02 = r0.z, a10 = r0.w, a11 = r1.x, a12 = r1.y, a20 = r1.z, a21 = r1.w,
                a22 = r2.x;
    const float D0 = r2.y, D1 = r2.z, D2 = r2.w;
    const float y0 = a00 * xx + a01 * xy + a02 * xz;
    const float y1 = a10 * xx + a11 * xy + a12 * xz;
    const float y2 = a20 * xx + a21 * xy + a22 * xz;
    const float e0 = a00 * ray.dx + a01 * ray.dy + a02 * ray.dz;
    const float e1 = a10 * ray.dx + a11 * ray.dy + a12 * ray.dz;
    const float e2 = a20 * ray.dx + a21 * ray.dy + a22 * ray.dz;
    // R^T ((o - m) x d) = y x e: a rotation preserves cross products
    const float v0 = y1 * e2 - y2 * e1;
    const float v1 = y2 * e0 - y0 * e2;
    const float v2 = y0 * e1 - y1 * e0;
    const float o0 = D0 * y0, o1 = D1 * y1, o2 = D2 * y2;
    const float d0 = D0 * e0, d1 = D1 * e1, d2 = D2 * e2;
    const float u0 = (D1 * D2) * v0, u1 = (D0 * D2) * v1, u2 = (D0 * D1) * v2;
    const float a = d0 * d0 + d1 * d1 + d2 * d2;
    const float b = o0 * d0 + o1 * d1 + o2 * d2;
    const float uu = u0 * u0 + u1 * u1 + u2 * u2;
    const float ia = __builtin_amdgcn_rcpf(a);
    G = HitGeom{y0, y1, y2, e0, e1, e2, u0, u1, u2, b, ia};
    return uu * ia;
}

// Second part: the nearer root t1 (meaningful where h2 <= Q). Both root forms are computed for
// every lane and one is selected, no divergent branch (where the ray hits the chosen form is
// the same arithmetic).
__device__ inline float ellipsoid_t1(const HitGeom &G, const float4 r2, float h2, float Q)
{
    const float D0 = r2.y, D1 = r2.z, D2 = r2.w;
    const float o0 = D0 * G.y0, o1 = D1 * G.y1, o2 = D2 * G.y2;
    const float sq = __builtin_amdgcn_sqrtf((Q - h2) * G.ia);  // hardware square root (1 ulp)
    const float tc = -G.b * G.ia;
    const float oo = o0 * o0 + o1 * o1 + o2 * o2;
    const float t_viete = ((oo - Q) * G.ia) * __builtin_amdgcn_rcpf(tc + sq);
    float t1 = G.b >= 0.0f ? tc - sq : t_viete;
    if (t1 == 0.0f) t1 = 0.0f;  // -0 -> +0 so the key order matches float order
    return t1;
}

__device__ inline bool ellipsoid_hit(const Ray &ray, const float4 r0, const float4 r1, const float4 r2, const float4 r3,
                                     float Q, float &t1, float &h2, HitGeom &G)
{
    h2 = ellipsoid_h2(ray, r0, r1, r2, r3, G);
    t1 = ellipsoid_t1(G, r2, h2, Q);
    return h2 <= Q;
}

// ------------------------------------------------------------- hit buffer

// A hit's sort key (t1, Gaussian index) packed into the bit pattern of a
// positive normal double: ((float bits of t1) + 2^20) << 32 | index. For
// t1 >= 0 the double order is the (t1, index) order, so a sorted insert is a
// chain of v_min_f64 / v_max_f64 (no compares, selects or hazards).
constexpr uint32_t kKeyBias = 0x00100000u;  // keeps every key a normal double
constexpr double kNoHit = __builtin_huge_val();  // empty slot, above every key

__device__ inline double hit_key(float t1, uint32_t gid)
{
    const uint64_t hi = uint64_t(__float_as_uint(t1) + kKeyBias);
    return __longlong_as_double((long long)((hi << 32) | gid));
}
__device__ inline float hit_key_t(double k)
{
    return __uint_as_float(uint32_t(uint64_t(__double_as_longlong(k)) >> 32) - kKeyBias);
}
__device__ inline uint32_t hit_key_gid(double k) { return uint32_t(uint64_t(__double_as_longlong(k))); }

// The smallest key of depth t >= 0 (any real key with t1 < t lies below it, any other above or at it;
// a key of t1 = +inf or NaN lies above it for t = +inf, one of a negative t1 below every such key).
__device__ inline double bound_key(float t) { return hit_key(t, 0u); }

// Sorted insert of k into the ascending keys key[0..N): slot s becomes max(key[s-1],
// min(key[s], k)) and slot 0 min(key[0], k), each from the old keys, so the 2N operations do
// not form a chain through a carried key. They are issued from the back, each max three slots
// behind its min, so a min's result is read five instructions later (f64 results need wait
// states before they are read; two slots behind left some). The keys are never NaN, so the
// min/max are the bare instructions (the generic fmin/fmax would first quiet every key in IEEE
// mode). OUT: returns max(key[N-1], k), the key pushed out (else kNoHit).
template <int N, bool OUT>
__device__ inline double sorted_insert(double (&key)[N], double k)
{
    double out = kNoHit;
    if (OUT) asm volatile("v_max_f64 %0, %1, %2" : "=v"(out) : "v"(key[N - 1]), "v"(k));
    double t[N];
#pragma unroll
    for (int s = N - 1; s >= -2; --s) {
        if (s >= 0) asm volatile("v_min_f64 %0, %1, %2" : "=v"(t[s]) : "v"(key[s]), "v"(k));
        const int m = s + 3;  // the slot whose max is due
        if (m >= 1 && m <= N - 1) asm volatile("v_max_f64 %0, %1, %2" : "=v"(key[m]) : "v"(key[m - 1]), "v"(t[m]));
    }
    key[0] = t[0];
    return out;
}

template <int K>
struct HitBuf {
    static constexpr int size = K;
    double key[K];  // sorted ascending; kNoHit marks an empty slot

    __device__ inline void clear()
    {
#pragma unroll
        for (int s = 0; s < K; ++s) key[s] = kNoHit;
    }
    __device__ inline double front() const { return key[0]; }
    __device__ inline double last() const { return key[K - 1]; }

    // drop the front entry (static register moves: no dynamic indexing)
    __device__ inline void pop_front()
    {
#pragma unroll
        for (int s = 0; s + 1 < K; ++s) key[s] = key[s + 1];
        key[K - 1] = kNoHit;
    }

    // sorted insert of k; the last entry falls off (inserting kNoHit changes nothing). The keys
    // are never NaN, so the min/max are the bare instructions: the generic fmin/fmax would first
    // quiet every loop-carried key (one more v_max_f64 per entry in IEEE mode).
    __device__ inline void insert(double k) { sorted_insert<K, false>(key, k); }
    // the same, returning the key that falls off (kNoHit: none)
    __device__ inline double insert_out(double k) { return sorted_insert<K, true>(key, k); }
};

// The same sorted buffer of KR + KT keys with its last KT entries in LDS: a per-wave ring of KT
// slots of 64 lanes (slot-major, so one slot of the wave is one contiguous 512-byte row) whose
// wave-uniform head is the tail's first entry. The registers hold the KR smallest keys. An
// insertion runs the register chain, then carries its key on through the tail when some lane
// carries one; a pop shifts the registers and takes the tail's first entry into the last one.
// `kmax` mirrors the buffer's last entry, so the candidate test and the culling bound need no
// LDS read. The workgroup is one wave.
#ifndef RS_RING_GROUP
#define RS_RING_GROUP 8
#endif
template <int KR, int KT>
struct HitBufTail {
    static constexpr int size = KR + KT;
    double key[KR];
    double kmax;
    int32_t head;
    double *ring;  // this wave's LDS ring, KT x 64 doubles
    int lane;

    __device__ inline void clear()
    {
#pragma unroll
        for (int s = 0; s < KR; ++s) key[s] = kNoHit;
        kmax = kNoHit;
        head = 0;
#pragma unroll
        for (int i = 0; i < KT; ++i) ring[i * kWave + lane] = kNoHit;
    }
    __device__ inline double front() const { return key[0]; }
    __device__ inline double last() const { return kmax; }

    __device__ inline void pop_front()
    {
#pragma unroll
        for (int s = 0; s + 1 < KR; ++s) key[s] = key[s + 1];
        double *e = ring + head * kWave + lane;
        key[KR - 1] = *e;
        *e = kNoHit;
        head = head + 1 == KT ? 0 : head + 1;
        kmax = kNoHit;
    }

    __device__ inline void insert(double k)
    {
        k = sorted_insert<KR, true>(key, k);
        if (!wave_ballot(k != kNoHit)) return;  // every carried key fell into an empty register slot
        // the ring's entries are read RG at a time (their LDS reads in flight together), then
        // passed through the min/max chain and written back
        constexpr int RG = RS_RING_GROUP;
        static_assert(KT % RG == 0, "ring group");
        int32_t p = head;
#pragma unroll
        for (int g = 0; g < KT; g += RG) {
            double t[RG];
            double *e[RG];
#pragma unroll
            for (int i = 0; i < RG; ++i) {
                e[i] = ring + p * kWave + lane;
                p = p + 1 == KT ? 0 : p + 1;
            }
#pragma unroll
            for (int i = 0; i < RG; ++i) t[i] = *e[i];
#pragma unroll
            for (int i = 0; i < RG; ++i) {
                double hi = 0.0;
                if (g + i + 1 < KT) asm volatile("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(t[i]), "v"(k));
                asm volatile("v_min_f64 %0, %0, %1" : "+v"(t[i]) : "v"(k));
                if (g + i + 1 == KT) kmax = t[i];
                k = hi;
            }
#pragma unroll
            for (int i = 0; i < RG; ++i) *e[i] = t[i];
        }
    }
};

// The forward's buffer for a hit-buffer size K. At K = 48 the last 16 keys live in LDS (8 KB
// per wave): 32 keys in registers let the kernel run four waves per SIMD instead of three,
// which hides more of the node and record fetch latency than the LDS traffic of the tail costs
// (measured: 9.6 against 10.5 ms at the scene-scale workload; 28 + 20 keys 9.7, 36 + 12 9.6,
// 40 + 8 10.3). At K = 32 the same split loses (16 + 16 keys at five waves: 10.5 against 10.3).
constexpr int kTailKeys = 16;
template <int K>
struct FwdBuf {
    using type = HitBuf<K>;
};
template <>
struct FwdBuf<48> {
    using type = HitBufTail<48 - kTailKeys, kTailKeys>;
};

// ------------------------------------------------------------- compositing

// One front-to-back step (Eq. 3): shared by the forward and adjoint kernels so
// both see bit-identical T and C sequences.
struct Accum {
    float T, Cr, Cg, Cb;
    int n;
};

__device__ inline void composite_step(Accum &A, float a, float cr, float cg, float cb)
{
    const float w = A.T * a;
    A.Cr = __builtin_fmaf(w, cr, A.Cr);
    A.Cg = __builtin_fmaf(w, cg, A.Cg);
    A.Cb = __builtin_fmaf(w, cb, A.Cb);
    const float om = 1.0f - a;
    A.T = A.T * om;
    A.n += 1;
}

__device__ inline bool stop_after(const Accum &A, const RenderParams &P)
{
    return A.T < P.eps1 || (P.max_hits > 0 && A.n >= P.max_hits);
}

// --------------------------------------------------------------- adjoint

// Gradient of h^2 (and so of alpha = opacity exp(-h^2/2)) for one hit, in the
// Gaussian's body frame. With p = o' - (b/a) d' (the whitened closest point,
// obtained without cancellation as p = (d' x u) / a, u = o' x d'), D = diag(1/s)
// and y_w = y - (b/a) e the body-frame closest-approach offset, App. A.6 gives
//   dh2/dm = -2 R D p,   dh2/ds_k = -2 D_k p_k^2,   dh2/dR = 2 R y_w (D p)^T.
// The rotation enters only through R^T dh2/dR, whose antisymmetric part is the
// angular vector w = 2 (D p) x y_w: a change dR = R [dtheta]x changes h2 by
// <w, dtheta>. So a hit contributes, per Gaussian,
//   acc_m = gh D p,  acc_s = -2 gh D_k p_k^2,  acc_w = 2 gh (D p) x y_w,
// (gh = dL/dh2), and k_scatter_grads applies R and the quaternion map once per
// Gaussian: dL/dm = -2 R acc_m, dL/dq = (2/|q|) E(q/|q|)^T acc_w, where
// dtheta = (2/|q|) E(n) dq, E(n) = [-v | w I - [v]x] for n = (w, v).
struct GradOut {
    float v[13];  // mean (body frame) 3, scale 3, angular 3, opacity 1, rgb 3
};

__device__ inline void grad_hit(const float4 r2, const HitGeom &g, float h2, float dLda, float alpha, GradOut &G)
{
    const float D0 = r2.y, D1 = r2.z, D2 = r2.w;
    const float d0 = D0 * g.e0, d1 = D1 * g.e1, d2 = D2 * g.e2;
    // p = (d' x u) / a
    const float p0 = (d1 * g.u2 - d2 * g.u1) * g.ia;
    const float p1 = (d2 * g.u0 - d0 * g.u2) * g.ia;
    const float p2 = (d0 * g.u1 - d1 * g.u0) * g.ia;
    const float Dp0 = D0 * p0, Dp1 = D1 * p1, Dp2 = D2 * p2;
    const float ba = g.b * g.ia;
    const float w0 = g.y0 - ba * g.e0, w1 = g.y1 - ba * g.e1, w2 = g.y2 - ba * g.e2;
    const float gh = dLda * (-0.5f * alpha);  // dL/dh2
    G.v[0] = gh * Dp0;
    G.v[1] = gh * Dp1;
    G.v[2] = gh * Dp2;
    G.v[3] = gh * (-2.0f * Dp0 * p0);
    G.v[4] = gh * (-2.0f * Dp1 * p1);
    G.v[5] = gh * (-2.0f * Dp2 * p2);
    const float c = 2.0f * gh;
    G.v[6] = c * (Dp1 * w2 - Dp2 * w1);
    G.v[7] = c * (Dp2 * w0 - Dp0 * w2);
    G.v[8] = c * (Dp0 * w1 - Dp1 * w0);
    // opacity: alpha = opacity * exp(-h2/2)
    G.v[9] = dLda * __expf(-0.5f * h2);
}

// ----------------------------------------------------------------- kernel

// One set of rays traced by a launch: its rays, optional per-ray limit and
// background, outputs (forward) or upstream gradient (adjoint), and its state.
struct RaySet {
    const float *origin, *dir, *tmax, *bgray, *grad;
    float *out_rgb;
    float4 *fin;  // final colour and T
    uint4 *last;  // last composited key, restart point of the T recursion
    int4 *list;   // stored-list bookkeeping (hit lists only)
    float bg[3];
    int32_t zero_colour;
};

struct Ptrs {
    const float *rgb;
    RaySet set[kMaxSets];
    int32_t *status;
    uint32_t *queue;  // XCD queue counters (kXcdQueues)
    unsigned long long *counters;
    float *gacc;  // adjoint accumulator, 16 floats per Gaussian (see k_scatter_grads)
    ListPool pool;
};

// ------------------------------------------------------- shared kernel steps

// Next packet of a wave (wave-uniform; n_packets when there is none). Plain
// grids take one packet per workgroup; persistent ones first drain the queue
// of their own XCD's chunk (a compact image region, so that XCD's L2 holds
// its working set), then take from the other chunks.
#ifndef RS_XCD_RUN
#define RS_XCD_RUN 32
#endif
constexpr int64_t kXcdRun = RS_XCD_RUN;

template <typename PT>
__device__ inline int64_t next_packet(const PT &P, uint32_t *queue, int lane, int xcd, int &qi, int64_t &iter)
{
    if (!P.persistent) {
        // plain grid: workgroups are dealt to the XCDs in turn, so workgroup b runs on XCD
        // b mod 8. Packets are dealt in runs of kXcdRun consecutive ones (a compact strip of
        // tiles), so the waves an XCD runs at a time share fewer Gaussians in its L2, while
        // every XCD still samples the whole image (the grid is rounded up to whole deals; the
        // few packets beyond n_packets exit)
        if (iter++ > 0) return P.n_packets;
        const int64_t b = blockIdx.x, i = b / kXcdQueues;
        return (i / kXcdRun * kXcdQueues + b % kXcdQueues) * kXcdRun + i % kXcdRun;
    }
    while (qi < kXcdQueues) {
        const int q = (xcd + qi) & (kXcdQueues - 1);
        uint32_t p = 0;
        if (lane == 0) p = atomicAdd(queue + q, 1u);
        p = __builtin_amdgcn_readfirstlane(p);
        const int64_t g = q * P.chunk + p;
        if (g < P.n_packets && p < P.chunk) return g;
        ++qi;
    }
    return P.n_packets;
}

__device__ inline int xcd_id() { return int(__builtin_amdgcn_s_getreg(20 | (0 << 6) | ((4 - 1) << 11))) & (kXcdQueues - 1); }

// A lane's ray of packet `pkt`: its set, index, geometry, t_max and background.
struct LaneRay {
    int si;
    bool valid;
    int64_t id;
    Ray ray;
    float tmax, bgr, bgg, bgb;
};

template <typename PT>
__device__ inline LaneRay lane_ray(const PT &P, const Ptrs &ptr, int64_t pkt, int lane)
{
    LaneRay L;
    L.si = 0;
    while (L.si + 1 < kMaxSets && pkt >= int64_t(L.si + 1) * P.packets_per_set) ++L.si;
    const RaySet &S = ptr.set[L.si];
    const int64_t local = pkt - L.si * P.packets_per_set;
    L.id = packet_ray(P, P.persistent ? strip_major_packet(P, local, P.strip_tiles) : local, lane, L.valid);
    L.tmax = kInf;
    L.bgr = S.bg[0];
    L.bgg = S.bg[1];
    L.bgb = S.bg[2];
    if (L.valid) {
        L.ray.ox = S.origin[3 * L.id];
        L.ray.oy = S.origin[3 * L.id + 1];
        L.ray.oz = S.origin[3 * L.id + 2];
        L.ray.dx = S.dir[3 * L.id];
        L.ray.dy = S.dir[3 * L.id + 1];
        L.ray.dz = S.dir[3 * L.id + 2];
        if (S.tmax) L.tmax = S.tmax[L.id];
        if (S.bgray) {
            L.bgr = S.bgray[3 * L.id];
            L.bgg = S.bgray[3 * L.id + 1];
            L.bgb = S.bgray[3 * L.id + 2];
        }
    } else {
        L.ray.ox = L.ray.oy = L.ray.oz = 0.0f;
        L.ray.dx = L.ray.dy = 0.0f;
        L.ray.dz = 1.0f;
    }
    return L;
}

// One composited hit (Eq. 3): the record of Gaussian gid is fetched, alpha is
// recomputed with the leaf test's own arithmetic (so every kernel sees the
// same alpha bit for bit) and the front-to-back step is applied.
struct HitData {
    float4 r0, r1, r2, r3;
    float al, cr, cg, cb, Tk;
    float t1, h2;  // entry distance (the hit key's t) and squared whitened distance
    HitGeom g;
};

// alpha of the Gaussian at sorted position js along the ray, with the leaf test's own arithmetic
__device__ inline float hit_alpha_at(int32_t js, const Ray &ray, const float4 *__restrict__ records, float Q,
                                     float4 &r0, float4 &r1, float4 &r2, float4 &r3, float &t1, float &h2,
                                     HitGeom &G)
{
    r0 = records[4 * js + 0];
    r1 = records[4 * js + 1];
    r2 = records[4 * js + 2];
    r3 = records[4 * js + 3];
    ellipsoid_hit(ray, r0, r1, r2, r3, Q, t1, h2, G);
    return r3.w * __expf(-0.5f * h2);
}

// alpha, colour and test intermediates of a hit (no compositing). EVERY: every lane
// computes, the caller giving idle lanes a valid Gaussian index whose values it never
// uses, so no lane is masked off and nothing is zeroed first.
template <bool EVERY = false>
__device__ inline void recompute_hit_at(bool act, uint32_t gid, int32_t js, const Ray &ray,
                                        const float4 *__restrict__ records, const float *__restrict__ rgb, bool zc,
                                        float Q, HitData &H)
{
    H.Tk = 0.0f;
    if (!EVERY) {
        H.al = H.cr = H.cg = H.cb = H.t1 = H.h2 = 0.0f;
        H.g = HitGeom{};
    }
    if (EVERY || act) {
        H.al = hit_alpha_at(js, ray, records, Q, H.r0, H.r1, H.r2, H.r3, H.t1, H.h2, H.g);
        H.cr = H.cg = H.cb = 0.0f;
        if (!zc) {
            H.cr = rgb[3 * gid];
            H.cg = rgb[3 * gid + 1];
            H.cb = rgb[3 * gid + 2];
        }
    }
}

// ------------------------------------------------------- back-to-front adjoint

// Smallest normal float: below it T loses relative precision, so the adjoint does not
// divide back from there (the forward saves the T before the hit that crossed it).
constexpr float kMinNormal = 1.17549435e-38f;

// Upstream gradient of a lane's pixel.
struct LaneGrad {
    float gr, gg, gb;
};

// Back-to-front state of a lane's adjoint: T_{k+1} (the transmittance behind
// the hit being processed), the colour S_{k+1} seen behind it (background
// first), the hits done so far, and where the forward's T fell below the normal
// floats: the T just before that hit (Tz) and how many composited hits followed
// it (mz, -1 when T stayed normal). Behind that hit T is taken as 0 (it is below
// 1.2e-38 there).
struct Back {
    float T, Sr, Sg, Sb, Tz;
    int32_t done, mz;
};

__device__ inline Back back_init(const float4 fin, const uint4 last, float bgr, float bgg, float bgb)
{
    Back B;
    B.T = fin.w;
    B.Sr = bgr;
    B.Sg = bgg;
    B.Sb = bgb;
    B.Tz = __uint_as_float(last.z);
    B.mz = int32_t(last.w);
    B.done = 0;
    return B;
}

// T_k of the next hit (back to front) with opacity al: T_{k+1} / (1 - al), except
// 0 behind the hit that took T below the normal floats and the saved T at that hit
// (a select, so a quotient 0/0 there is never used).
__device__ inline float back_T(const Back &B, float al)
{
    const float Td = B.T * __builtin_amdgcn_rcpf(1.0f - al);
    return B.done < B.mz ? 0.0f : (B.done == B.mz ? B.Tz : Td);
}

// hit k (alpha al, colour c) now lies behind the next hit: S <- al c + (1 - al) S
__device__ inline void back_over(Back &B, float al, float cr, float cg, float cb)
{
    B.Sr = __builtin_fmaf(al, cr - B.Sr, B.Sr);
    B.Sg = __builtin_fmaf(al, cg - B.Sg, B.Sg);
    B.Sb = __builtin_fmaf(al, cb - B.Sb, B.Sb);
}

// Per-wave gradient accumulation in LDS (the traversal adjoint): a table of Gaussian slots,
// each holding the 13 partial sums of one Gaussian, found by hashing its index with linear
// probing over kAccProbes slots. Every hit adds its values into its Gaussian's slot with LDS
// atomics; a slot's sums reach the global accumulators (one 64-byte line per Gaussian) only
// when the table is flushed: when some lane finds no slot in its probe window, and at the end
// of the kernel. The hits of one Gaussian on the rays of a packet, over every compositing
// step, so cost one line of global atomics per flush instead of one per step. The workgroup
// is one wave.
constexpr int kAccSlots = 128;
constexpr int kAccProbes = 8;
constexpr int kAccVals = 13;
struct AccTable {
    int32_t tag[kAccSlots];           // Gaussian index, -1: free
    int32_t list[kAccSlots];          // occupied slots, compacted by a flush
    float acc[kAccSlots * kAccVals];  // partial sums (odd stride: distinct slots, distinct banks)
};

__device__ inline AccTable &acc_table()
{
    __shared__ AccTable T;
    return T;
}

__device__ inline void acc_clear(AccTable &T, int lane)
{
    for (int s = lane; s < kAccSlots; s += kWave) T.tag[s] = -1;
    for (int s = lane; s < kAccSlots * kAccVals; s += kWave) T.acc[s] = 0.0f;
    __syncthreads();
}

__device__ inline uint32_t acc_home(uint32_t gid)
{
    return uint32_t((uint64_t(gid * 2654435761u) * uint64_t(kAccSlots)) >> 32);
}

// Adds every occupied slot's sums to the global accumulators (16-lane segments, one slot
// each, lane v of a segment adding value v) and frees the table.
template <bool COUNT>
__device__ inline void acc_flush(AccTable &T, float *gacc, int lane, uint64_t &c_group)
{
    __syncthreads();
    int32_t cnt = 0;
    for (int base = 0; base < kAccSlots; base += kWave) {
        const int s = base + lane;
        const bool occ = s < kAccSlots && T.tag[s] != -1;
        const uint64_t m = wave_ballot(occ);
        if (occ) T.list[cnt + int32_t(__builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u)))] = s;
        cnt += __popcll(m);
    }
    __syncthreads();
    const int v = lane & 15, q = lane >> 4;
    for (int i = 0; i < cnt; i += 4) {
        const int k = i + q;
        if (k < cnt && v < kAccVals) {
            const int s = T.list[k];
            const uint32_t g = uint32_t(T.tag[s]);
            float *a = T.acc + s * kAccVals + v;
            unsafeAtomicAdd(gacc + 16 * int64_t(g) + v, *a);
            *a = 0.0f;
        }
    }
    if (COUNT) c_group += uint64_t(cnt);
    __syncthreads();
    for (int s = lane; s < kAccSlots; s += kWave) T.tag[s] = -1;
    __syncthreads();
}

// One step of the pairwise sum: lanes paired by the DPP pattern CTRL (an involution) that
// hold the same Gaussian are merged into the `keep` lane of the pair. Called with every lane
// of the wave active.
template <int CTRL>
__device__ inline void acc_pair(bool &act, uint32_t gid, GradOut &G, bool keep)
{
    const int32_t pg = __builtin_amdgcn_mov_dpp(int32_t(gid), CTRL, 0xF, 0xF, false);
    const int32_t pa = __builtin_amdgcn_mov_dpp(act ? 1 : 0, CTRL, 0xF, 0xF, false);
    const bool m = act && pa != 0 && pg == int32_t(gid);
#pragma unroll
    for (int v = 0; v < kAccVals; ++v) {
        const float pv = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(G.v[v]), CTRL, 0xF, 0xF, false));
        G.v[v] = (m && keep) ? G.v[v] + pv : G.v[v];
    }
    act = act && !(m && !keep);
}

// Adjoint of one composited hit (App. A.3-A.6) and its wave aggregation.
//   dL/dalpha_k = T_k <g, c_k - S_{k+1}>,  dL/dc_k = alpha_k T_k g,
// then alpha's chain rule (grad_hit). TABLE: the contributions go into the wave's LDS table
// (the traversal adjoint, whose long traversal hides the LDS atomics). Otherwise (the stored-
// list adjoint, where the table's same-address LDS atomics would be the bottleneck) the active
// lanes' contributions are summed per distinct Gaussian of this step through LDS, and one
// 13-lane segment of an atomic instruction adds each Gaussian's totals to its 64-byte
// accumulator line (four Gaussians per instruction).
template <bool COUNT, bool TABLE>
__device__ inline void adjoint_hit(bool act, uint64_t act_mask, uint32_t gid, const HitData &H, float Tk,
                                   const Back &B, const LaneGrad &Gd, bool zc, float *gacc, int lane, uint64_t &c_group)
{
    GradOut G;
    // the table path sums neighbouring lanes' values, so idle lanes contribute zeros; the
    // stored-list path stores active lanes' values only and computes on every lane
    if (TABLE) {
#pragma unroll
        for (int v = 0; v < 13; ++v) G.v[v] = 0.0f;
    }
    if (!TABLE || act) {
        const float dLda = Tk * (Gd.gr * (H.cr - B.Sr) + Gd.gg * (H.cg - B.Sg) + Gd.gb * (H.cb - B.Sb));
        grad_hit(H.r2, H.g, H.h2, dLda, H.al, G);
        const float wgt = H.al * Tk;
        G.v[10] = zc ? 0.0f : Gd.gr * wgt;
        G.v[11] = zc ? 0.0f : Gd.gg * wgt;
        G.v[12] = zc ? 0.0f : Gd.gb * wgt;
    }
    if constexpr (TABLE) {
        (void)act_mask;
        // Lanes of one 16-lane row holding the same Gaussian are first summed pairwise (lane^1,
        // lane^2, then mirrored halves and rows: neighbouring pixels of the packet tile), so
        // fewer LDS atomics meet at one address.
        acc_pair<0xB1>(act, gid, G, (lane & 1) == 0);   // quad_perm [1,0,3,2]
        acc_pair<0x4E>(act, gid, G, (lane & 2) == 0);   // quad_perm [2,3,0,1]
        acc_pair<0x141>(act, gid, G, (lane & 7) < 4);   // row_half_mirror
        acc_pair<0x140>(act, gid, G, (lane & 15) < 8);  // row_mirror
        AccTable &T = acc_table();
        const uint32_t home = acc_home(gid);
        bool pend = act;
        for (;;) {
            int32_t slot = -1;
            if (pend) {
                uint32_t h = home;
                for (int p = 0; p < kAccProbes; ++p) {
                    const int32_t old = atomicCAS(&T.tag[h], -1, int32_t(gid));
                    if (old == -1 || old == int32_t(gid)) {
                        slot = int32_t(h);
                        break;
                    }
                    h = h + 1 == uint32_t(kAccSlots) ? 0u : h + 1;
                }
            }
            if (slot >= 0) {
                float *a = T.acc + slot * kAccVals;
#pragma unroll
                for (int v = 0; v < kAccVals; ++v)
                    __hip_atomic_fetch_add(a + v, G.v[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                pend = false;
            }
            // lanes left without a slot: flush the table and probe again from their home slots
            if (!wave_ballot(pend)) break;
            acc_flush<COUNT>(T, gacc, lane, c_group);
        }
    } else {
        // Lanes holding the same Gaussian form a group; groups are numbered in order of their
        // lowest lane and each group's lanes store their 13 values in consecutive LDS rows. The
        // scalar loop keeps only masks and counts in scalar registers; a lane records its row,
        // and after the loop each group's lowest lane writes the group's (Gaussian, first row),
        // the next group's first row closing it. Then 16-lane segments sum one
        // group's rows each, so one atomic instruction adds the totals of four Gaussians (one
        // 64-byte accumulator line per segment). The wave is the whole workgroup, and its LDS
        // operations complete in order.
        __shared__ float rows[kWave * 16];
        __shared__ int2 groups[kWave + 1];  // Gaussian index, first row
        uint64_t todo = act_mask, leaders = 0;
        int32_t pos = 0, mypos = 0;
        while (todo) {
            const int leader = __builtin_ctzll(todo);
            const uint32_t lg = __builtin_amdgcn_readlane(gid, leader);
            const uint64_t same = wave_ballot(gid == lg) & todo;
            const bool mine = __builtin_amdgcn_inverse_ballot_w64(same);  // this lane is in the group
            todo &= ~same;
            leaders |= 1ull << leader;
            if (COUNT) ++c_group;
            const int32_t at = int32_t(
                __builtin_amdgcn_mbcnt_hi(uint32_t(same >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(same), uint32_t(pos))));
            mypos = mine ? at : mypos;
            pos += __popcll(same);
        }
        const int32_t ng = __popcll(leaders);
        // a group's number is the number of leaders below its leader (groups open in lane order)
        const int32_t mygrp = int32_t(
            __builtin_amdgcn_mbcnt_hi(uint32_t(leaders >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(leaders), 0u)));
        if (__builtin_amdgcn_inverse_ballot_w64(leaders)) groups[mygrp] = make_int2(int32_t(gid), mypos);
        if (lane == 0) groups[ng] = make_int2(0, pos);
        if (act) {
            float *r = rows + 16 * mypos;
#pragma unroll
            for (int v = 0; v < 13; ++v) r[v] = G.v[v];
        }
        // the segments read other lanes' rows and descriptors: a (one-wave) barrier keeps the
        // compiler from reusing a lane's own earlier stores in their place
        __syncthreads();
        const int v = lane & 15;
        for (int b = 0; b < ng; b += 4) {
            const int gi = b + (lane >> 4);
            if (gi < ng && v < 13) {
                const int2 gd = groups[gi];
                const int32_t end = groups[gi + 1].y;
                float t = rows[16 * gd.y + v];
                for (int j = gd.y + 1; j < end; ++j) t += rows[16 * j + v];
                unsafeAtomicAdd(gacc + 16 * int64_t(uint32_t(gd.x)) + v, t);
            }
        }
    }
}

// ------------------------------------------------------------ stored lists

// Row cursor of a packet's stored list (wave-uniform).
struct ListCursor {
    int32_t rows;   // rows stored
    int32_t chunk;  // current chunk (-1: none yet)
    int32_t fill;   // slots used in the current chunk
    int32_t slots;  // slots stored (rows and masks)
    int32_t spare;  // last chunk of an abandoned attempt of this packet, its chunks to be used again (-1: none)
    bool ok;        // false once the pool was found exhausted
};

// Ends a block that only some lanes run, before wave-uniform values meet again: without it the
// compiler folds the block's end into the next join, takes that join's values for divergent and
// keeps them, and every branch on them, per lane.
__device__ inline void rejoin() { __builtin_amdgcn_wave_barrier(); }

// Ends a row whose steps took the lanes `mask`: its masks as two words.
__device__ inline void list_end_row(const ListPool &pool, ListCursor &L, uint64_t mask, int lane)
{
    uint32_t *end = pool.slots + int64_t(L.chunk) * pool.chunk_slots + L.fill;
    if (lane == 0) {
        __builtin_nontemporal_store(uint32_t(mask), end);
        __builtin_nontemporal_store(uint32_t(mask >> 32), end + 1);
    }
    rejoin();
    L.fill += 2;
    L.slots += 2;
    ++L.rows;
}

// steps in a row of a 16-ray packet, from its masks
__device__ inline int32_t row_steps(uint64_t mask) { return (79 - __builtin_clzll(mask)) >> 4; }

// Whether a row is one step. ROWS: steps in a row, 0: the pool says (read at run time, it cost the frontier's 64-ray
// packets 1.5 % with mirrors over 500,000 Gaussians, 22.1 against 21.8 ms a forward; known when compiled, 21.95).
template <int ROWS>
__device__ inline bool one_step(const ListPool &pool)
{
    return ROWS == 1 || (ROWS == 0 && pool.chunk_slots == kChunkSlots);
}

// Appends one step (called from wave-uniform control flow): the entries of the lanes whose `entry` is not
// kListIdle, in lane order. The masks of the open row of a 16-ray packet wait in `open` (LDS: in registers
// they would cost every packet). A row ends after kRowSteps steps, or where the next step and the masks
// do not fit the current chunk: that one starts a new chunk, taken from the pool
// and linked to the packet's previous chunk. Once the pool is exhausted the packet
// stores nothing more (the adjoint then traverses for its rays, or, for the paper
// variant, the sticky status reports it).
template <int ROWS>
__device__ inline void list_append(const ListPool &pool, ListCursor &L, uint64_t &open, uint32_t entry, int lane,
                                   bool paper, int32_t *status)
{
    const uint64_t m = wave_ballot(entry != kListIdle);
    if (m == 0) return;
    const int32_t k = __popcll(m);
    const bool wide = one_step<ROWS>(pool);
    uint64_t mask = 0;
    if (!wide)
        mask = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int32_t(open >> 32)))) << 32) |
               uint32_t(__builtin_amdgcn_readfirstlane(int32_t(open)));
    if (L.chunk < 0 || L.fill + k + 2 > pool.chunk_slots) {
        if (mask) list_end_row(pool, L, mask, lane);
        mask = 0;
        int32_t c = L.spare, spare = -1;
        if (lane == 0) {
            if (L.chunk >= 0) pool.fill[L.chunk] = L.fill;
            if (c >= 0) {
                spare = pool.prev[c];
            } else {
                const unsigned long long at = atomicAdd(pool.hdr, 1ull);
                c = at < (unsigned long long)pool.chunks ? int32_t(at) : -1;
            }
        }
        rejoin();
        c = __builtin_amdgcn_readfirstlane(c);
        L.spare = __builtin_amdgcn_readfirstlane(spare);
        if (c < 0) {
            L.ok = false;
            if (lane == 0) {
                atomicOr(pool.hdr + 1, 1ull);
                if (paper) atomicOr(status, kStatusListPool);
            }
            rejoin();
            return;
        }
        if (lane == 0) pool.prev[c] = L.chunk;
        rejoin();
        L.chunk = c;
        L.fill = 0;
    }
    // The rows are streamed out with nontemporal stores: they are read back only by the adjoint,
    // after this launch, and the forward's own fetches wait less behind them.
    uint32_t *row = pool.slots + int64_t(L.chunk) * pool.chunk_slots + L.fill;
    if (entry != kListIdle) {
        const uint32_t below = __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
        __builtin_nontemporal_store(entry, row + below);
    }
    if (wide) {
        if (lane == 0) {
            __builtin_nontemporal_store(uint32_t(m), row + k);
            __builtin_nontemporal_store(uint32_t(m >> 32), row + k + 1);
        }
        rejoin();
        L.fill += k + 2;
        L.slots += k + 2;
        ++L.rows;
        return;
    }
    rejoin();
    L.fill += k;
    L.slots += k;
    const int32_t step = mask ? row_steps(mask) : 0;
    mask |= m << (16 * step);
    if (step + 1 == kRowSteps) {
        list_end_row(pool, L, mask, lane);
        mask = 0;
    }
    open = mask;  // every lane the same word
}

// Ends the packet's last row and records the fill of its last chunk.
template <int ROWS>
__device__ inline void list_close(const ListPool &pool, ListCursor &L, uint64_t open, int lane)
{
    if (!one_step<ROWS>(pool) && L.ok && L.chunk >= 0 && wave_ballot(open != 0)) list_end_row(pool, L, open, lane);
    if (L.ok && L.chunk >= 0 && lane == 0) pool.fill[L.chunk] = L.fill;
}

// min of two floats that are never NaN-signalling, as the bare instruction
__device__ inline float fmin_bare(float a, float b)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

constexpr int32_t kDone = INT32_MIN;

// Wave-uniform descent from `node` through internal nodes to the next leaf
// (returned as ~leaf) or to the end of the walk (kDone). A child is entered
// when some live lane's ray overlaps its box within [t_lo, t_hi]; when both
// are, the one the leader lane reaches first (REV: leaves last) is taken and the
// other pushed (stack entry k lives in lane k of `stackv`). Ordering by the leader
// lane costs one compare instead of a vote and, in simulation at the scene-scale
// workload, visits within 0.5 % as many nodes as a majority vote. The loop has one exit (a
// full stack ends the walk through the same path as an empty one) and decides the
// two-children case with one scalar compare, which keeps the scalar control flow short.
template <int OCT, bool COUNT, bool REV>
__device__ inline int32_t descend(int32_t node, const float4 *__restrict__ nodes, const Slab &sl, uint64_t lead_bit,
                                  float t_lo, float t_hi_w, int lane, int32_t stack_depth, int32_t &sp,
                                  int32_t &stackv, bool &overflow, uint64_t &c_node, uint64_t &c_lchild)
{
    while (node >= 0) {
        const uint32_t ns = __builtin_amdgcn_readfirstlane(node);
        const float4 *nd = nodes + 4 * uint64_t(ns);
        const float4 n0 = nd[0], n1 = nd[1], n2 = nd[2];
        const int2 lr = *reinterpret_cast<const int2 *>(nd + 3);
        float ln, lf, rn, rf;
        child_slabs<OCT>(n0, n1, n2, sl, ln, lf, rn, rf);
        // [max(near, t_lo), min(widened exit, t_hi)] non-empty as two compares against
        // x = min(widened exit, t_hi): t_lo <= t_hi holds on every live lane, and t_lo is NaN on
        // the others, so no compare passes there. The min is the bare instruction (t_hi is
        // loop-carried; the generic fminf would quiet it first).
        const float lx = fmin_bare(widen_exit(lf, sl.pad), t_hi_w), rx = fmin_bare(widen_exit(rf, sl.pad), t_hi_w);
        const uint64_t bl = wave_ballot(ln <= lx) & wave_ballot(t_lo <= lx);
        const uint64_t br = wave_ballot(rn <= rx) & wave_ballot(t_lo <= rx);
        const int32_t left = lr.x, right = lr.y;
        if (COUNT) {
            ++c_node;
            c_lchild += __popcll(bl) + __popcll(br);
        }
        // nonzero iff both children are entered (one scalar compare for the branch)
        const uint32_t both = min(uint32_t(__popcll(bl)), uint32_t(__popcll(br)));
        int32_t next;
        if (both != 0) {
            // both entered: the child the leader lane (lowest live lane) reaches first (REV: leaves
            // last) goes first
            const bool lfirst = (wave_ballot(REV ? lf >= rf : ln <= rn) & lead_bit) != 0;
            if (sp >= stack_depth) {
                overflow = true;
                next = kDone;
            } else {
                stackv = (lane == sp) ? (lfirst ? right : left) : stackv;
                ++sp;
                next = lfirst ? left : right;
            }
        } else if ((bl | br) != 0) {
            next = bl != 0 ? left : right;
        } else if (sp == 0) {
            next = kDone;
        } else {
            --sp;
            next = __builtin_amdgcn_readlane(stackv, sp);
        }
        node = next;
    }
    return node;
}

// The wave-uniform walk of the whole BVH for one round: descend to a leaf, test it
// (leaf(j), which may move t_lo / t_hi_w), resume from the stack. The walk is specialised on the
// wave's direction octant as a whole, so the octant is dispatched once per walk.
#define RS_WALK_OCT(O)                                                                                        \
    {                                                                                                         \
        int32_t node = P.root;                                                                                \
        int32_t sp = 0;                                                                                       \
        int32_t stackv = 0;                                                                                   \
        const uint64_t live_mask = wave_ballot(live);                                                         \
        const uint64_t lead_bit = live_mask & (~live_mask + 1);                                               \
        for (;;) {                                                                                            \
            node = descend<O, COUNT, kRev>(node, nodes, sl, lead_bit, t_lo, t_hi_w, lane, P.stack_depth, sp,  \
                                           stackv, overflow, c_node, c_lchild);                               \
            if (node == kDone) break;                                                                         \
            leaf(~node);                                                                                      \
            if (sp == 0) break;                                                                               \
            --sp;                                                                                             \
            node = __builtin_amdgcn_readlane(stackv, sp);                                                     \
        }                                                                                                     \
    }

#define RS_WALK_BVH()                                                                                         \
    switch (oct) {                                                                                            \
    case 0: RS_WALK_OCT(0) break;                                                                             \
    case 1: RS_WALK_OCT(1) break;                                                                             \
    case 2: RS_WALK_OCT(2) break;                                                                             \
    case 3: RS_WALK_OCT(3) break;                                                                             \
    case 4: RS_WALK_OCT(4) break;                                                                             \
    case 5: RS_WALK_OCT(5) break;                                                                             \
    case 6: RS_WALK_OCT(6) break;                                                                             \
    case 7: RS_WALK_OCT(7) break;                                                                             \
    default: RS_WALK_OCT(kMixedOctant) break;                                                                 \
    }

// Occupancy target (waves per SIMD) of each variant, i.e. its VGPR budget
// (512 / waves): the adjoint carries the gradient temporaries as well. The
// forward targets are measured optima: a few dozen bytes of scratch spills
// (kbuf 24 at five waves, 48 at four with its LDS tail) cost less than the
// node-fetch latency the extra wave hides, while larger spills (kbuf 24 at six,
// 32 at five) lose.
// The adjoint's are measured the same way: kbuf 24 and 32 at four waves and
// 48 at three beat one wave fewer by 10-20 %, while one wave more (five, and
// four for 48) spills heavily and doubles the time.
#ifndef RS_FWD16_WAVES
#define RS_FWD16_WAVES 5
#endif
#ifndef RS_BWD16_WAVES
#define RS_BWD16_WAVES 4
#endif
#ifndef RS_FWD24_WAVES
#define RS_FWD24_WAVES 5
#endif
#ifndef RS_BWD24_WAVES
#define RS_BWD24_WAVES 4
#endif
#ifndef RS_BWD32_WAVES
#define RS_BWD32_WAVES 4
#endif
#ifndef RS_BWD48_WAVES
#define RS_BWD48_WAVES 3
#endif
#ifndef RS_FWD32_WAVES
#define RS_FWD32_WAVES 4
#endif
#ifndef RS_FWD48_WAVES
#define RS_FWD48_WAVES 4
#endif
constexpr int waves_for(int K, bool bwd)
{
    return bwd ? (K <= 8 ? 4 : (K <= 16 ? RS_BWD16_WAVES : (K <= 24 ? RS_BWD24_WAVES : (K <= 32 ? RS_BWD32_WAVES : RS_BWD48_WAVES))))
               : (K <= 8 ? 6 : (K <= 16 ? RS_FWD16_WAVES : (K <= 24 ? RS_FWD24_WAVES : (K <= 32 ? RS_FWD32_WAVES : RS_FWD48_WAVES))));
}

// ------------------------------------------------------------ forward render

// A lane's ray while its packet is traced: the front-to-back accumulator, and with
// RS_PAPER_GRADIENT its second phase: after an eps1 stop the lane keeps consuming hits without
// compositing them, recording their ids while T2 (their transmittance) stays >= eps2.
struct LaneState {
    Ray ray;
    Accum A;
    bool live;
    double last;  // the last consumed key
    bool phase2;
    float T2;
    int32_t extra;
};

// What a lane seldom writes lives in LDS: T just before the composited hit that took T below the
// normal floats (to 0, or into the subnormals, where T_{k+1} / (1 - alpha_k) would lose its digits)
// and that hit's index, and how many composited ids were stored when the list pool ran out. And the lane masks of
// the open list row.
struct LaneCold {
    float Tz[kWave];
    int32_t z[kWave], stored[kWave];
    uint64_t open;
};

template <int ROWS>
__device__ inline void lane_reset(LaneState &S, LaneCold &C, bool live, int lane)
{
    S.A = Accum{1.0f, 0.0f, 0.0f, 0.0f, 0};
    S.live = live;
    S.last = -kNoHit;
    S.phase2 = false;
    S.T2 = 1.0f;
    S.extra = 0;
    C.Tz[lane] = 0.0f;
    C.z[lane] = -1;
    if (ROWS != 1) C.open = 0;
}

// One compositing step of the wave: the lanes with `act` consume their hit `key`, of opacity al and
// colour c.
template <bool PAPER, int ROWS>
__device__ inline void consume_known(bool act, double key, float al, float cr, float cg, float cb, LaneState &S,
                                     LaneCold &C, const Ptrs &ptr, const RenderParams &P, bool lists, ListCursor &LC,
                                     int lane)
{
    const bool paper = PAPER && P.paper && lists;
    const uint32_t gid = hit_key_gid(key);
    uint32_t entry = kListIdle;
    if (paper && S.phase2) {
        if (act) {
            if (S.T2 < P.eps2 || S.A.n + S.extra >= P.max_hits) {
                S.live = false;  // the second phase ends before this hit
            } else {
                entry = gid | kListSecond;
                S.T2 *= 1.0f - al;
                ++S.extra;
                S.last = key;
            }
        }
    } else {
        const float Tk = S.A.T;
        if (act) {
            composite_step(S.A, al, cr, cg, cb);
            entry = gid;
            S.last = key;
            if (S.A.T < kMinNormal && Tk >= kMinNormal) {
                C.Tz[lane] = Tk;
                C.z[lane] = S.A.n - 1;
            }
        }
        const bool stopped = act && stop_after(S.A, P);
        if (stopped) {
            if (paper && S.A.T < P.eps1)
                S.phase2 = true;  // stays live for the second phase
            else
                S.live = false;
        }
        rejoin();
    }
    if (lists && LC.ok) {
        list_append<ROWS>(ptr.pool, LC, C.open, entry, lane, paper, ptr.status);
        if (!LC.ok) C.stored[lane] = S.A.n - (entry < kListSecond ? 1 : 0);
    }
    rejoin();
}

// The same with the hit's opacity and colour fetched here (Gaussian at sorted position js): alpha is
// recomputed from the record with the leaf test's own arithmetic.
template <bool PAPER, int ROWS>
__device__ inline void consume(bool act, double key, int32_t js, LaneState &S, LaneCold &C,
                               const float4 *__restrict__ records, const Ptrs &ptr, const RenderParams &P, bool zc,
                               bool lists, ListCursor &LC, int lane)
{
    float al = 0.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
    if (act) {
        float4 r0, r1, r2, r3;
        float t1, h2;
        HitGeom hg;
        al = hit_alpha_at(js, S.ray, records, P.Q, r0, r1, r2, r3, t1, h2, hg);
        if (!zc) {
            const uint32_t gid = hit_key_gid(key);
            cr = ptr.rgb[3 * int64_t(gid)];
            cg = ptr.rgb[3 * int64_t(gid) + 1];
            cb = ptr.rgb[3 * int64_t(gid) + 2];
        }
    }
    rejoin();
    consume_known<PAPER, ROWS>(act, key, al, cr, cg, cb, S, C, ptr, P, lists, LC, lane);
}

// The outputs and the adjoint's starting state of a packet's rays.
template <int ROWS>
__device__ inline void write_rays(const LaneState &S, const LaneCold &C, const LaneRay &LR, const RaySet &R,
                                  const Ptrs &ptr, ListCursor &LC, bool lists, int lane)
{
    if (lists) list_close<ROWS>(ptr.pool, LC, C.open, lane);
    if (!LR.valid) return;
    const float orr = __builtin_fmaf(S.A.T, LR.bgr, S.A.Cr), og = __builtin_fmaf(S.A.T, LR.bgg, S.A.Cg),
                ob = __builtin_fmaf(S.A.T, LR.bgb, S.A.Cb);
    R.out_rgb[3 * LR.id] = orr;
    R.out_rgb[3 * LR.id + 1] = og;
    R.out_rgb[3 * LR.id + 2] = ob;
    if (R.fin) {
        R.fin[LR.id] = make_float4(orr, og, ob, S.A.T);
        const uint64_t kb = S.A.n > 0 ? uint64_t(__double_as_longlong(S.last)) : 0ull;
        const int32_t z = C.z[lane];
        R.last[LR.id] = make_uint4(uint32_t(kb), uint32_t(kb >> 32), __float_as_uint(C.Tz[lane]),
                                   z >= 0 ? uint32_t(S.A.n - 1 - z) : 0xffffffffu);
    }
    if (lists) R.list[LR.id] = make_int4(S.A.n, LC.ok ? S.A.n : C.stored[lane], LC.chunk, LC.rows);
}

// Work counters of a forward wave (wave-uniform; only in the COUNT variants).
struct FwdCount {
    uint64_t pkt, node, leaf, round, lleaf, lbuf, lcomp, lchild, rows, slots;
};
__device__ inline void add_counts(const FwdCount &c, const Ptrs &ptr, int lane)
{
    if (lane != 0 || c.pkt == 0) return;
    atomicAdd(ptr.counters + 0, (unsigned long long)c.pkt);
    atomicAdd(ptr.counters + 1, (unsigned long long)c.node);
    atomicAdd(ptr.counters + 2, (unsigned long long)c.leaf);
    atomicAdd(ptr.counters + 3, (unsigned long long)c.round);
    atomicAdd(ptr.counters + 4, (unsigned long long)c.lleaf);
    atomicAdd(ptr.counters + 5, (unsigned long long)c.lbuf);
    atomicAdd(ptr.counters + 6, (unsigned long long)c.lcomp);
    atomicAdd(ptr.counters + 7, (unsigned long long)c.lchild);
    atomicAdd(ptr.counters + 12, (unsigned long long)c.rows);
    atomicAdd(ptr.counters + 14, (unsigned long long)c.slots);
}

// The depth-first walk of a packet, in rounds, until no lane is live. Returns false when the traversal
// stack overflowed.
template <typename BUF, bool BRUTE, bool COUNT, bool PAPER, int ROWS>
__device__ inline bool walk_rounds(LaneState &S, LaneCold &C, const LaneRay &LR, bool zc, bool lists, ListCursor &LC,
                                   const float4 *__restrict__ records, const float4 *__restrict__ nodes,
                                   const int32_t *__restrict__ gidx, const int32_t *__restrict__ inv, const Ptrs &ptr,
                                   const RenderParams &P, BUF &hb, int lane, FwdCount &cnt)
{
    constexpr bool kRev = false;
    const Ray &ray = S.ray;
    const float tmax = LR.tmax;
    bool &live = S.live;
    const Slab sl = make_slab(ray);
    const int oct = wave_octant(sl, LR.valid);
    bool overflow = false;
    uint64_t c_node = 0, c_lchild = 0;
    while (wave_ballot(live)) {
        hb.clear();
        if (COUNT) ++cnt.round;
        const double last = S.last;
        // NaN on lanes that are not live: no box test passes for them
        const float t_lo =
            !live ? __builtin_nanf("") : (last == -kNoHit ? P.t_min : fmaxf(P.t_min, hit_key_t(last)));
        float t_hi_w = widen(tmax, sl.pad);

        // the round's live lanes as a mask: the leaf step combines per-compare masks with it
        // (a ballot of a compound condition would first turn it into a vector value)
        const uint64_t live_now = wave_ballot(live);
        auto leaf = [&](int64_t j) {
            const int64_t js = __builtin_amdgcn_readfirstlane(int32_t(j));
            const float4 r0 = records[4 * js + 0], r1 = records[4 * js + 1], r2 = records[4 * js + 2],
                         r3 = records[4 * js + 3];
            const uint32_t gid = uint32_t(gidx[js]);
            // every lane evaluates the test and the key (no divergent branch); only lanes
            // whose ray hits take part, and the entry distance and key only when one does
            HitGeom hg;
            const float h2 = ellipsoid_h2(ray, r0, r1, r2, r3, hg);
            // the index load is issued with the record's (its latency hides behind theirs)
            asm volatile("" ::"s"(gid));
            if (COUNT) {
                ++cnt.leaf;
                cnt.lleaf += __popcll(live_now);
            }
            const uint64_t hmask = wave_ballot(h2 <= P.Q) & live_now;
            if (!hmask) return;
            const float t1 = ellipsoid_t1(hg, r2, h2, P.Q);
            const double k = hit_key(t1, gid);
            const uint64_t cmask = hmask & wave_ballot(t1 >= P.t_min) & wave_ballot(t1 < tmax) &
                                   wave_ballot(k > last) & wave_ballot(k < hb.last());
            const bool cand = __builtin_amdgcn_inverse_ballot_w64(cmask);
            if (COUNT) cnt.lbuf += __popcll(cmask);
            if (cmask) {
                // every lane runs the insertion network; lanes without a candidate insert
                // the empty key, which moves nothing
                hb.insert(cand ? k : kNoHit);
                if (hb.last() != kNoHit) t_hi_w = widen(fminf(tmax, hit_key_t(hb.last())), sl.pad);
            }
        };

        if (BRUTE) {
            for (int64_t j = 0; j < P.n_gauss; ++j) leaf(j);
        } else {
            // While-while traversal: descend internal nodes until a leaf is reached (or the
            // stack runs dry), then test that leaf; the hit buffer changes only in the leaf step.
            RS_WALK_BVH()
        }
        if (overflow) {
            live = false;
            return false;
        }

        // composite this round's hits front to back; the buffer is consumed from its front
        const double round_last = hb.last();
        bool more = true;
        // the sorted position of the buffer's front key is looked up one step ahead, so its
        // latency overlaps the previous step (an empty key reads position 0, unused)
        int32_t js_next = inv[hb.front() != kNoHit ? hit_key_gid(hb.front()) : 0u];
#pragma unroll 1
        for (int s = 0; s < hb.size; ++s) {
            const double key_s = hb.front();
            const int32_t js_s = js_next;
            hb.pop_front();
            js_next = inv[hb.front() != kNoHit ? hit_key_gid(hb.front()) : 0u];
            const bool act = more && live && key_s != kNoHit;
            const uint64_t act_mask = wave_ballot(act);
            more = act_mask != 0;
            if (!more) break;
            if (COUNT) cnt.lcomp += __popcll(act_mask);
            consume<PAPER, ROWS>(act, key_s, js_s, S, C, records, ptr, P, zc, lists, LC, lane);
        }
        // a lane whose buffer did not fill has consumed all its hits
        if (live && round_last == kNoHit) live = false;
    }
    if (COUNT) {
        cnt.node += c_node;
        cnt.lchild += c_lchild;
    }
    return true;
}

// The walk as a kernel of its own: for brute force, for calls that bound the traversal stack, and for the paper
// variant, whose pool is sized for the walk's rows: every step consumes a hit of each live ray, so a packet stores at
// most max_hits of them. (The frontier drains its rays at different steps: up to four times as many rows.)
template <int K, bool BRUTE, bool COUNT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(waves_for(K, false)))) void k_render(
    const float4 *__restrict__ records, const float4 *__restrict__ nodes, const int32_t *__restrict__ gidx,
    const int32_t *__restrict__ inv, const Ptrs ptr, const RenderParams P)
{
    const int lane = threadIdx.x;
    int64_t iter_pkt = 0;
    const int xcd = xcd_id();
    int qi = 0;
    FwdCount cnt{};
    for (;;) {
        const int64_t pkt = next_packet(P, ptr.queue, lane, xcd, qi, iter_pkt);
        if (pkt >= P.n_packets) break;
        if (COUNT) ++cnt.pkt;
        const LaneRay LR = lane_ray(P, ptr, pkt, lane);
        const RaySet &R = ptr.set[LR.si];
        const bool zc = R.zero_colour != 0;
        const bool lists = P.lists && R.list != nullptr;
        ListCursor LC{0, -1, 0, 0, -1, true};
        __shared__ LaneCold cold;
        LaneState S;
        S.ray = LR.ray;
        lane_reset<0>(S, cold, LR.valid && P.n_gauss > 0 && LR.tmax > P.t_min, lane);
        typename FwdBuf<K>::type hb;
        if constexpr (!std::is_same<typename FwdBuf<K>::type, HitBuf<K>>::value) {
            __shared__ double ring[kTailKeys * kWave];
            hb.ring = ring;
            hb.lane = lane;
        }
        if (!walk_rounds<typename FwdBuf<K>::type, BRUTE, COUNT, true, 0>(S, cold, LR, zc, lists, LC, records, nodes, gidx, inv, ptr,
                                                                       P, hb, lane, cnt))
            if (lane == 0) atomicOr(ptr.status, kStatusStack);
        write_rays<0>(S, cold, LR, R, ptr, LC, lists, lane);
        if (COUNT) {
            cnt.rows += uint64_t(LC.rows);
            cnt.slots += uint64_t(LC.slots);
        }
    }
    if (COUNT) add_counts(cnt, ptr, lane);
}

// ------------------------------------------------------- frontier forward
//
// The depth-first walk visits a node with the whole wave, one dependent 64-byte fetch per visit,
// tests every leaf that some ray's box interval meets, and starts again from the root for the rays
// with more hits than the buffer holds. The frontier kernel turns the search round: the lanes test
// 64 nodes (or 64 leaves) at a time against the bundle of the packet's rays, in windows of depth
// from near to far, and only the leaves that survive are tested ray by ray, in order of a lower
// bound of their depth. So a hit that is nearer than every leaf still to come is final: it is
// composited and leaves the buffer at once, a packet visits each leaf once, and stops where its
// rays do.
//
// Depth is measured along z, the coordinate axis (with a sign) that a packet's rays run along: z0
// is the smallest origin, and a ray is u = a_u + z m_u, v = a_v + z m_v over z >= 0, so the bundle
// is bounded by the extremes of a and m (the four planes of a frustum for rays of one origin).
// A node is dropped when its box misses the bundle; a leaf when its ellipsoid does (its support
// against the four planes) or when it misses the tube around the bundle's centre line.
//
// The result is the walk's bit for bit as long as no bound is too tight: a leaf that the bundle drops is not
// tested, and a lane that has stopped looks for no nearer hit. So the bounds carry margins for the
// rounding of the ray test (kFrontMargin of a depth, Bundle::pad of a length: camera and scene at 1, 50 and 1000 units
// from the coordinate origin, one ray to sixteen, along an axis or not, some 50 million hits, four fifths of them on
// flat Gaussians near their rim: none dropped, none in front of its bound). The rest does not hang on them:
// a lane whose buffer overflows remembers the smallest key it lost (`cap`), takes no hit beyond it and is traced
// again from its last consumed key, and a hit found after a later one was consumed makes the packet start over
// with the walk.

constexpr int kFrontActive = 256;  // nodes to expand in this window
constexpr int kFrontNodes = 192;   // nodes beyond this window
constexpr int kFrontLeaves = 384;  // leaves tested against the bundle, of this window and beyond
constexpr int kFrontSorted = 192;  // leaves tested ray by ray per window at most
constexpr int kFrontRaw = 128;     // leaves found, not yet tested
constexpr int kFrontWindows = 1 << 14, kFrontRounds = 4096;  // windows of a round, rounds of a packet: then the walk
constexpr float kFrontFirst = 1.0f;     // Gaussians held that the first window is made for (0.5: 5.7, 1.5: 5.3 ms at 1M; 1.5, 1.8 at 100k)
// Gaussians a bundle may hold, by volume; beyond that the packet is walked, since a bundle that spans much of the
// scene drops little of it. (500k Gaussians, 4 x 1024x768 with mirrors: 22 ms at 512 to 2048, 144 at 4096, 34 when all
// is walked; 1M, 320x180 with lists: 9.6, 6.2 and 5.2 ms at 512, 2048 and 4096.) A walk costs less the smaller the
// scene, so the bound is a share of it too. (30k, 320x240 with a mirror and shadows: 1.4 ms walked from 469 on, 15.8
// from 2048 on.)
constexpr float kFrontHeld = 2048.0f, kFrontHeldLeast = 256.0f, kFrontShare = 1.0f / 64.0f;
// A frontier also gives way to the walk while it is at work, which the volume alone does not foresee:
// - where most leaves that it tests ray by ray are hit by none: after kFrontTested pairs, when under a quarter had a hit
//   (the case above, were it not for its volume: 98 % without a hit, 50000 leaves);
// - where many rays need many rounds, each of them searched from the root: the walk shares its visits among the
//   rays that are left, a frontier of few rays is narrow. Rounds, and rays left, of 64-ray packets and of smaller ones:
//   10k large translucent Gaussians, 640x480: 10.3 ms (11.5 in the frontier, 10.9 walked); 3k: 7.0 (10.0, 7.6);
//   500k, 640x361 with mirrors: 10.6 (19.5, 10.5); 1M, 1920x1080: 4.8 (5.3, 7.8). With 24 rays left after three rounds
//   100k, 800x800 takes 1.9 ms (1.6); 16-ray packets after four rounds with eight left: 1M, 320x180 with lists 6.8
//   (5.8 here). Launches of several sets give way sooner: reflected and shadow rays spread (500k, 160x120 with a
//   mirror and shadows, lists: 9.4 ms; 15.7 after eight rounds, 16.6 walked, 30 in the frontier).
constexpr int kFrontTested = 256;
constexpr int kWideRounds = 4, kWideLeft = 24, kSmallRounds = 8, kSmallLeft = 14, kSetsRounds = 2, kSetsLeft = 4;
constexpr float kFrontBack = 4e-3f;       // of the depth from which a later round tests boxes, relative
constexpr float kFrontMargin = 1.2e-4f;  // of a depth bound, relative: the rounding of t1 of flat ellipsoids

struct FrontLds {
    double start[kWave], stop[kWave];  // a lane's keys lie between them in this round, and in all
    float from[kWave];                 // depth from which hits are left
    int32_t ar[kFrontActive];
    float nz[kFrontNodes];
    int32_t nr[kFrontNodes];
    float pz[kFrontLeaves];
    int32_t pr[kFrontLeaves];
    float sz[kFrontSorted];
    int32_t sr[kFrontSorted];
    int32_t raw[kFrontRaw];
    uint32_t hist[kWave];
};

// Wave-wide minimum and sums by DPP: row shifts, then broadcasts across the rows of 16 lanes; the
// last lane holds the result. A lane without a source keeps its own value.
template <int CTRL, int ROWS>
__device__ inline float dpp_min(float x)
{
    const float y = __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), CTRL, ROWS, 0xF, false));
    return fminf(x, y);
}
__device__ inline float wave_min(float x)
{
    x = dpp_min<0x111, 0xF>(x);  // row_shr 1, 2, 4, 8
    x = dpp_min<0x112, 0xF>(x);
    x = dpp_min<0x114, 0xF>(x);
    x = dpp_min<0x118, 0xF>(x);
    x = dpp_min<0x142, 0xA>(x);  // row_bcast 15 into rows 1 and 3
    x = dpp_min<0x143, 0xC>(x);  // row_bcast 31 into rows 2 and 3
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), kWave - 1));
}
__device__ inline float wave_max(float x) { return -wave_min(-x); }

__device__ inline uint32_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
}

// A wave-uniform value in a scalar register: vector registers are what the frontier is short of.
__device__ inline float uniform(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }

// A packet's axes and ray bundle (wave-uniform but for the lane's own ozr, dz).
struct Bundle {
    int ax;      // axis of z; u and v are the next two
    float sg;    // +1: z along the axis, -1: against it
    float z0;    // smallest origin (in z)
    float Au0, Au1, Mu0, Mu1, Av0, Av1, Mv0, Mv1;
    float ru0, ru1, rv0, rv1;  // 1 / M
    float zfrom, zlo, zhi;  // hits are wanted from zfrom (zlo for boxes) to zhi
    float rq;        // sqrt(Q)
    float pad;       // absolute slack: rounding at the scale of the origins and of the scene
};

__device__ inline float pick(int ax, float x, float y, float z) { return ax == 0 ? x : (ax == 1 ? y : z); }

// Bounds of the rays of the lanes with `on`; (ozr, dz): the lane's origin beyond z0 and its direction
// along z, so z(t) = ozr + t dz.
__device__ inline void bundle_bounds(Bundle &B, const Ray &ray, bool on, float ozr, float dz)
{
    const float iz = 1.0f / dz;
    const float mu = pick(B.ax, ray.dy, ray.dz, ray.dx) * iz, mv = pick(B.ax, ray.dz, ray.dx, ray.dy) * iz;
    const float au = pick(B.ax, ray.oy, ray.oz, ray.ox) - ozr * mu, av = pick(B.ax, ray.oz, ray.ox, ray.oy) - ozr * mv;
    constexpr float s = 4e-6f;
    auto lo = [&](float x) { const float m = wave_min(on ? x : kInf); return m - s * fabsf(m); };
    auto hi = [&](float x) { const float m = wave_max(on ? x : -kInf); return m + s * fabsf(m); };
    B.Mu0 = lo(mu);
    B.Mu1 = hi(mu);
    B.Mv0 = lo(mv);
    B.Mv1 = hi(mv);
    B.Au0 = lo(au) - B.pad;
    B.Au1 = hi(au) + B.pad;
    B.Av0 = lo(av) - B.pad;
    B.Av1 = hi(av) + B.pad;
    // a slope of 0 counts as leaving the box (the lower line rising, the upper one falling), so that
    // its test is that of A alone
    auto slope = [](float m, float none) { return fabsf(m) > 1e-30f ? m : none; };
    B.Mu0 = slope(B.Mu0, 1e-30f);
    B.Mu1 = slope(B.Mu1, -1e-30f);
    B.Mv0 = slope(B.Mv0, 1e-30f);
    B.Mv1 = slope(B.Mv1, -1e-30f);
    B.ru0 = 1.0f / B.Mu0;
    B.ru1 = 1.0f / B.Mu1;
    B.rv0 = 1.0f / B.Mv0;
    B.rv1 = 1.0f / B.Mv1;
}

// Whether a box meets the bundle: the depths at which the bundle lies inside each pair of its planes,
// met with [zlo, zhi]. Its depth bound (with margin) in `near`. The bundle's lower line u = A0 + z M0
// must lie below the box's upper plane, its upper line above the lower plane: each holds from a depth
// on (the line runs toward the box) or up to one.
__device__ inline bool box_meets(const Bundle &B, float lx, float ly, float lz, float hx, float hy, float hz, float &near)
{
    const float l = pick(B.ax, lx, ly, lz), h = pick(B.ax, hx, hy, hz);
    const float lu = pick(B.ax, ly, lz, lx), hu = pick(B.ax, hy, hz, hx);
    const float lv = pick(B.ax, lz, lx, ly), hv = pick(B.ax, hz, hx, hy);
    const float za = (B.sg > 0.0f ? l : -h) - B.z0, zb = (B.sg > 0.0f ? h : -l) - B.z0;
    const float qu0 = (hu - B.Au0) * B.ru0, qu1 = (lu - B.Au1) * B.ru1;
    const float qv0 = (hv - B.Av0) * B.rv0, qv1 = (lv - B.Av1) * B.rv1;
    float enter = fmaxf(fmaxf(za, 0.0f), B.Mu0 < 0.0f ? qu0 : 0.0f);
    enter = fmaxf(fmaxf(enter, B.Mu1 > 0.0f ? qu1 : 0.0f), fmaxf(B.Mv0 < 0.0f ? qv0 : 0.0f, B.Mv1 > 0.0f ? qv1 : 0.0f));
    float exit = fminf(zb, B.Mu0 < 0.0f ? kInf : qu0);
    exit = fminf(fminf(exit, B.Mu1 > 0.0f ? kInf : qu1), fminf(B.Mv0 < 0.0f ? kInf : qv0, B.Mv1 > 0.0f ? kInf : qv1));
    near = fmaxf(__builtin_fmaf(enter, -kFrontMargin, enter) - B.pad, B.zlo);
    exit = __builtin_fmaf(fabsf(exit), kFrontMargin, exit) + B.pad;
    return near <= exit && near <= B.zhi;
}

// Whether the ellipsoid of a record can meet a ray of the bundle, and a lower bound of the depth of
// any hit (with margin). Written so that NaN keeps the leaf.
__device__ inline bool ellipsoid_meets(const Bundle &B, float Q, const float4 r0, const float4 r1, const float4 r2,
                                       const float4 r3, float &near)
{
    const float a[3][3] = {{r0.x, r0.y, r0.z}, {r0.w, r1.x, r1.y}, {r1.z, r1.w, r2.x}};
    const float D[3] = {r2.y, r2.z, r2.w};
    float Z[3], U[3], V[3], s[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        Z[k] = B.sg * pick(B.ax, a[k][0], a[k][1], a[k][2]);
        U[k] = pick(B.ax, a[k][1], a[k][2], a[k][0]);
        V[k] = pick(B.ax, a[k][2], a[k][0], a[k][1]);
        s[k] = __builtin_amdgcn_rcpf(D[k]);
    }
    const float mz = B.sg * pick(B.ax, r3.x, r3.y, r3.z) - B.z0, mu = pick(B.ax, r3.y, r3.z, r3.x),
                mv = pick(B.ax, r3.z, r3.x, r3.y);
    // support of the ellipsoid along the plane normal X - m Z
    auto support = [&](const float *X, float m) {
        float e = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float w = (X[k] - m * Z[k]) * s[k];
            e = __builtin_fmaf(w, w, e);
        }
        return __builtin_amdgcn_sqrtf(Q * e) * 1.0001f + B.pad;
    };
    bool out = (mu - B.Au1 - mz * B.Mu1) > support(U, B.Mu1);
    out = out || (B.Au0 + mz * B.Mu0 - mu) > support(U, B.Mu0);
    out = out || (mv - B.Av1 - mz * B.Mv1) > support(V, B.Mv1);
    out = out || (B.Av0 + mz * B.Mv0 - mv) > support(V, B.Mv0);
    float ez = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) ez = __builtin_fmaf(Z[k] * s[k], Z[k] * s[k], ez);
    ez = __builtin_amdgcn_sqrtf(Q * ez) * 1.0001f + B.pad;
    out = out || mz + ez < B.zlo;
    // the centre line against the ellipsoid grown by the tube's half widths at its far end: a hit at
    // depth z lies within delta (whitened) of the line's point at z
    const float cu = 0.5f * (B.Mu0 + B.Mu1), cv = 0.5f * (B.Mv0 + B.Mv1);
    const float zf = fmaxf(mz + ez, 0.0f);
    const float wu = 0.5f * ((B.Au1 - B.Au0) + zf * (B.Mu1 - B.Mu0)), wv = 0.5f * ((B.Av1 - B.Av0) + zf * (B.Mv1 - B.Mv0));
    const float xz = -mz, xu = 0.5f * (B.Au0 + B.Au1) - mu, xv = 0.5f * (B.Av0 + B.Av1) - mv;
    float y[3], e[3], g2 = 0.0f, gd = 0.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        y[k] = Z[k] * xz + U[k] * xu + V[k] * xv;
        e[k] = Z[k] + U[k] * cu + V[k] * cv;
        const float p = D[k] * U[k] * wu, q = D[k] * V[k] * wv;
        g2 += p * p + q * q;
        gd += p * q;
    }
    const float u0 = D[1] * D[2] * (y[1] * e[2] - y[2] * e[1]), u1 = D[0] * D[2] * (y[2] * e[0] - y[0] * e[2]),
                u2 = D[0] * D[1] * (y[0] * e[1] - y[1] * e[0]);
    const float d0 = D[0] * e[0], d1 = D[1] * e[1], d2 = D[2] * e[2];
    const float ia = __builtin_amdgcn_rcpf(d0 * d0 + d1 * d1 + d2 * d2);
    const float b = D[0] * y[0] * d0 + D[1] * y[1] * d1 + D[2] * y[2] * d2;
    const float hh = (u0 * u0 + u1 * u1 + u2 * u2) * ia;
    const float rr = B.rq + __builtin_amdgcn_sqrtf(g2 + 2.0f * fabsf(gd));
    const float disc = rr * rr * 1.001f - hh;
    out = out || disc < 0.0f;
    const float zc = -b * ia;
    // rounding of t1 (and of zc): an error of |x| ulp in y moves it by D / |d'| of that
    const float slack = 2e-7f * (fabsf(xz) + fabsf(xu) + fabsf(xv)) * fmaxf(fmaxf(D[0], D[1]), D[2]) *
                            __builtin_amdgcn_sqrtf(ia) + kFrontMargin * fabsf(zc) + B.pad;
    // A ray enters in front of its point nearest to the centre. With w the ray's (whitened) offset from
    // the line at zc and w1 its change per depth, that point lies (<q, w1> + <w, d' + w1>) / |d' + w1|^2
    // from zc, |q| <= rr, |w| <= delta, |w1| <= delta / zf; used where |w1| <= |d'| / 2
    const float delta = rr - B.rq, w1 = delta * __builtin_amdgcn_rcpf(zf);
    const float behind = 4.0f * rr * w1 * ia + 2.0f * delta * __builtin_amdgcn_sqrtf(ia);
    out = out || (w1 * w1 * ia <= 0.25f && zc + behind * 1.001f + slack < B.zfrom);
    // fmaxf returns the other operand for a NaN
    const float zn = fmaxf(mz - ez, zc - __builtin_amdgcn_sqrtf(disc * ia));
    near = fmaxf(zn - slack, B.zfrom);
    out = out || near > B.zhi;
    return !out;
}

// min of two keys (never NaN) as the bare instruction
__device__ inline double min_bare(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

constexpr int kFrontDrain = 32;  // lanes with a final hit that make a drain step worth while
constexpr int kFrontWaves = 4;  // per SIMD

// kNoHit made where it is used: as a constant of the whole kernel it is spilled, and each insertion waits
// for it (5 % of the frontier's time).
__device__ inline double no_hit_here()
{
    uint32_t lo, hi;
    asm volatile("v_mov_b32 %0, 0\n\tv_mov_b32 %1, 0x7ff00000" : "=&v"(lo), "=v"(hi));
    return __longlong_as_double((long long)((uint64_t(hi) << 32) | lo));
}

// ROWS: steps in a row of its stored lists (see list_append).
template <int K, bool COUNT, int ROWS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kFrontWaves))) void k_render_front(
    const float4 *__restrict__ records, const float4 *__restrict__ nodes, const int32_t *__restrict__ gidx,
    const int32_t *__restrict__ inv, const Ptrs ptr, const RenderParams P)
{
    __shared__ FrontLds F;
    __shared__ LaneCold cold;
    const int lane = threadIdx.x;
    int64_t iter_pkt = 0;
    const int xcd = xcd_id();
    int qi = 0;
    const float root_q = uniform(__builtin_amdgcn_sqrtf(P.Q)), closed_at = uniform(0.99f * P.eps1);
    FwdCount cnt{};
    for (;;) {
        const int64_t pkt = next_packet(P, ptr.queue, lane, xcd, qi, iter_pkt);
        if (pkt >= P.n_packets) break;
        if (COUNT) ++cnt.pkt;
        LaneState S;
        bool zc, lists;
        {
            const LaneRay LR = lane_ray(P, ptr, pkt, lane);
            S.ray = LR.ray;
            const bool wanted = LR.valid && P.n_gauss > 0 && LR.tmax > P.t_min;
            lane_reset<ROWS>(S, cold, wanted, lane);
            zc = ptr.set[LR.si].zero_colour != 0;
            lists = P.lists && ptr.set[LR.si].list != nullptr;
            // hits are taken with start < key < stop
            F.start[lane] = __longlong_as_double(__double_as_longlong(bound_key(P.t_min)) - 1);
            F.stop[lane] = bound_key(LR.tmax);
            F.from[lane] = P.t_min;
            S.last = F.start[lane];
        }
        ListCursor LC{0, -1, 0, 0, -1, true};
        HitBuf<K> hb;
        // A group that is better walked is left to the walk, which goes on behind the hits that its rays have
        // consumed; only where their order was wrong does the packet start over.
        bool leave = false, redo = false;
        // groups of rays along one axis (most packets are one group)
        uint64_t todo = wave_ballot(S.live);
        while (todo && !redo) {
            const int leader = __builtin_ctzll(todo);
            auto of_leader = [&](float x) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), leader)); };
            const float lx = of_leader(S.ray.dx), ly = of_leader(S.ray.dy), lz = of_leader(S.ray.dz);
            Bundle B;
            B.rq = root_q;
            B.ax = fabsf(lx) >= fabsf(ly) && fabsf(lx) >= fabsf(lz) ? 0 : (fabsf(ly) >= fabsf(lz) ? 1 : 2);
            B.sg = pick(B.ax, lx, ly, lz) >= 0.0f ? 1.0f : -1.0f;
            // the lane's direction and origin along z: z(t) = ozr + t dz
            auto dz_of = [&]() { return B.sg * pick(B.ax, S.ray.dx, S.ray.dy, S.ray.dz); };
            auto ozr_of = [&]() { return B.sg * pick(B.ax, S.ray.ox, S.ray.oy, S.ray.oz) - B.z0; };
            uint64_t grp;  // the group's rays
            {
                const float dz = dz_of();
                const float du = pick(B.ax, S.ray.dy, S.ray.dz, S.ray.dx), dv = pick(B.ax, S.ray.dz, S.ray.dx, S.ray.dy);
                grp = wave_ballot(fabsf(du) <= 2.0f * dz && fabsf(dv) <= 2.0f * dz) & todo & wave_ballot(S.live);
                if (!grp) break;  // a direction without a largest component (not a number)
                const bool on = __builtin_amdgcn_inverse_ballot_w64(grp);
                const float oz = B.sg * pick(B.ax, S.ray.ox, S.ray.oy, S.ray.oz);
                B.z0 = wave_min(on ? oz : kInf);
                B.pad = wave_max(on ? fabsf(S.ray.ox) + fabsf(S.ray.oy) + fabsf(S.ray.oz) : 0.0f);
            }
            // The ray test rounds in proportion to the offset between origin and mean, some 4e-7 of it
            auto reach_of = [](float x, float y) { return fmaxf(fabsf(x), fabsf(y)); };
            float held = 0.0f;  // Gaussians in the bundle, by volume
            if (P.root >= 0) {
                const float4 n0 = nodes[0], n1 = nodes[1], n2 = nodes[2];
                const float lx = fminf(n0.x, n1.z), ly = fminf(n0.y, n1.w), lz = fminf(n0.z, n2.x);
                const float hx = fmaxf(n0.w, n2.y), hy = fmaxf(n1.x, n2.z), hz = fmaxf(n1.y, n2.w);
                B.pad = uniform(2e-6f * fmaxf(B.pad, reach_of(lx, hx) + reach_of(ly, hy) + reach_of(lz, hz)));
                const float za = (B.sg > 0.0f ? pick(B.ax, lx, ly, lz) : -pick(B.ax, hx, hy, hz)) - B.z0;
                const float zb = (B.sg > 0.0f ? pick(B.ax, hx, hy, hz) : -pick(B.ax, lx, ly, lz)) - B.z0;
                const float eu = pick(B.ax, hy - ly, hz - lz, hx - lx), ev = pick(B.ax, hz - lz, hx - lx, hy - ly);
                const float dz = dz_of(), ozr = ozr_of(), idz = 1.0f / dz;
                const bool on = __builtin_amdgcn_inverse_ballot_w64(grp);
                const float reach = __builtin_fmaf(hit_key_t(F.stop[lane]), dz, ozr);
                const float z1 = fminf(zb, wave_max(on ? reach : 0.0f)), z0 = fmaxf(za, 0.0f);
                if (z1 > z0) {
                    // the bundle's cross-section at both ends of the scene
                    const float mu = pick(B.ax, S.ray.dy, S.ray.dz, S.ray.dx) * idz, mv = pick(B.ax, S.ray.dz, S.ray.dx, S.ray.dy) * idz;
                    const float au = pick(B.ax, S.ray.oy, S.ray.oz, S.ray.ox) - ozr * mu, av = pick(B.ax, S.ray.oz, S.ray.ox, S.ray.oy) - ozr * mv;
                    auto span = [&](float x) { return wave_max(on ? x : -kInf) - wave_min(on ? x : kInf); };
                    const float wu = fmaxf(span(au + z0 * mu), span(au + z1 * mu)), wv = fmaxf(span(av + z0 * mv), span(av + z1 * mv));
                    held = fminf(wu, eu) * fminf(wv, ev) * (z1 - z0) * float(P.n_gauss) / (eu * ev * (zb - za));
                }
            } else {
                const float4 r3 = records[3];
                B.pad = 2e-6f * fmaxf(B.pad, fabsf(r3.x) + fabsf(r3.y) + fabsf(r3.z));
            }
            todo &= ~grp;
            if (!(B.pad < 1e30f)) continue;  // an origin that is not finite: no bound holds for the others
            // rays that share little: most leaves of the bundle would be tested for nothing
            if (held > fminf(kFrontHeld, fmaxf(kFrontHeldLeast, kFrontShare * float(P.n_gauss)))) continue;
            leave = false;
            int rounds = 0, tested = 0, useful = 0;  // pairs of leaves tested ray by ray, and those that a ray hits
            // rounds, until the group's rays have stopped or run out of hits
            for (uint64_t on_mask = grp & wave_ballot(S.live); on_mask && !leave && !redo; on_mask = grp & wave_ballot(S.live)) {
                if (COUNT) ++cnt.round;
                hb.clear();
                double cap = F.stop[lane];
                F.start[lane] = S.last;
                rejoin();
                float Tv = S.A.T, tv = 0.0f;  // T behind every hit buffered so far, and the farthest one's depth
                const uint64_t began = on_mask;
                int nA = 0, nN = 0, nP = 0, nR = 0, n_on;
                {
                    const bool on = __builtin_amdgcn_inverse_ballot_w64(on_mask);
                    const float dz = dz_of(), ozr = ozr_of();
                    const float tl = F.from[lane];
                    const float zl = wave_min(on ? __builtin_fmaf(tl, dz, ozr) : kInf);
                    B.zfrom = uniform(fmaxf(zl - kFrontMargin * fabsf(zl) - B.pad, 0.0f));
                    B.zlo = uniform(fmaxf(zl - kFrontBack * fabsf(zl) - B.pad, 0.0f));
                    const float zh = wave_max(on ? __builtin_fmaf(hit_key_t(cap), dz, ozr) : -kInf);
                    B.zhi = uniform(zh + kFrontMargin * fabsf(zh) + B.pad);
                    bundle_bounds(B, S.ray, on, ozr, dz);
                    n_on = __popcll(on_mask);
                }
                float S0 = 0.0f, S1 = kInf, dS = kInf;  // the window [S0, S1)
                __syncthreads();
                if (P.root >= 0) {
                    const float4 n0 = nodes[0], n1 = nodes[1], n2 = nodes[2];
                    const float lx = fminf(n0.x, n1.z), ly = fminf(n0.y, n1.w), lz = fminf(n0.z, n2.x);
                    const float hx = fmaxf(n0.w, n2.y), hy = fmaxf(n1.x, n2.z), hz = fmaxf(n1.y, n2.w);
                    float near;
                    if (!box_meets(B, lx, ly, lz, hx, hy, hz, near)) near = kInf;
                    near = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(near)));
                    const float zf = (B.sg > 0.0f ? pick(B.ax, hx, hy, hz) : -pick(B.ax, lx, ly, lz)) - B.z0;
                    // the first window: the share of the root's depth range that may hold a window's leaves
                    // (boxes overlap a bundle that their centres are far from: some tens per Gaussian held)
                    if (near < kInf) {
                        F.ar[0] = P.root;
                        nA = 1;
                        S0 = near;
                        dS = fmaxf((zf - near) * fminf(fmaxf(kFrontFirst / fmaxf(held, 1e-3f), 1.0f / 64.0f), 0.125f),
                                   1e-5f * fabsf(zf) + 1e-20f);
                        S1 = S0 + dS;
                    }
                } else {
                    F.raw[0] = ~P.root;
                    nR = 1;
                }
                __syncthreads();

                // every window tests leaves or moves on; the bound on their number is a backstop
                int windows = 0;
                for (bool more = true; more;) {
                    if (++windows > kFrontWindows) {
                        leave = true;
                        break;
                    }
                    // ---- expand the window's nodes, and test the leaves found against the bundle
                    bool forced = false;  // the leaf pool ran full first
                    while (nA > 0 || nR > 0) {
                        if (nR >= kWave || nA == 0) {
                            if (nP > kFrontLeaves - kWave) {
                                forced = true;
                                break;
                            }
                            const int m = nR < kWave ? nR : kWave;
                            const int32_t js = F.raw[nR - m + (lane < m ? lane : 0)];
                            nR -= m;
                            const float4 r0 = records[4 * int64_t(js)], r1 = records[4 * int64_t(js) + 1],
                                         r2 = records[4 * int64_t(js) + 2], r3 = records[4 * int64_t(js) + 3];
                            float near;
                            const uint64_t km = wave_ballot(ellipsoid_meets(B, P.Q, r0, r1, r2, r3, near) && lane < m);
                            if (__builtin_amdgcn_inverse_ballot_w64(km)) {
                                const int at = nP + int(lanes_below(km));
                                F.pz[at] = near;
                                F.pr[at] = js;
                            }
                            nP += __popcll(km);
                            __syncthreads();
                            continue;
                        }
                        if (nA >= kFrontActive) {
                            leave = true;
                            break;
                        }
                        // children: at most 2 m more leaves and nodes
                        int m = nA < kWave ? nA : kWave;
                        const int room_r = (kFrontRaw - nR) / 2, room_a = (kFrontActive - nA + 1) / 2;
                        m = m < room_r ? m : room_r;
                        m = m < room_a ? m : room_a;
                        const bool mine = lane < m;
                        const int32_t node = F.ar[nA - m + (mine ? lane : 0)];
                        nA -= m;
                        const float4 *nd = nodes + 4 * int64_t(node);
                        const float4 n0 = nd[0], n1 = nd[1], n2 = nd[2];
                        const int2 lr = *reinterpret_cast<const int2 *>(nd + 3);
                        float ln, rn;
                        const uint64_t hl = wave_ballot(box_meets(B, n0.x, n0.y, n0.z, n0.w, n1.x, n1.y, ln) && mine);
                        const uint64_t hr = wave_ballot(box_meets(B, n1.z, n1.w, n2.x, n2.y, n2.z, n2.w, rn) && mine);
                        if (COUNT) {
                            cnt.node += m;
                            cnt.lchild += __popcll(hl) + __popcll(hr);
                        }
                        const bool full = nN > kFrontNodes - 2 * kWave;  // no room beyond the window: expand at once
                        __syncthreads();
#pragma unroll
                        for (int c = 0; c < 2; ++c) {
                            const uint64_t h = c ? hr : hl;
                            const int32_t ref = c ? lr.y : lr.x;
                            const float near = c ? rn : ln;
                            const uint64_t leafs = wave_ballot(ref < 0), now = full ? ~0ull : wave_ballot(near < S1);
                            const uint64_t mr = h & leafs, ma = h & ~leafs & now, mn = h & ~leafs & ~now;
                            if (__builtin_amdgcn_inverse_ballot_w64(mr)) F.raw[nR + int(lanes_below(mr))] = ~ref;
                            if (__builtin_amdgcn_inverse_ballot_w64(ma)) F.ar[nA + int(lanes_below(ma))] = ref;
                            if (__builtin_amdgcn_inverse_ballot_w64(mn)) {
                                const int at = nN + int(lanes_below(mn));
                                F.nz[at] = near;
                                F.nr[at] = ref;
                            }
                            rejoin();
                            nR += __popcll(mr);
                            nA += __popcll(ma);
                            nN += __popcll(mn);
                        }
                        __syncthreads();
                    }
                    if (leave) break;

                    // ---- the window's leaves in depth order: a counting sort over 64 depth bins
                    F.hist[lane] = 0u;
                    __syncthreads();
                    float take = S1;
                    if (forced) {
                        // the pool is full while nodes of the window are left: bins over all it holds
                        float far = S0;
                        for (int b = 0; b < nP; b += kWave)
                            if (b + lane < nP) far = fmaxf(far, F.pz[b + lane]);
                        take = wave_max(far) * 1.0001f + 1e-20f;
                        dS *= 0.25f;
                    }
                    const float wbin = take < kInf ? (take - S0) * (1.0f / 64.0f) : 0.0f;
                    const float inv_w = wbin > 0.0f ? 1.0f / wbin : 0.0f;
                    auto bin_of = [&](float z) { return int(fminf(fmaxf((z - S0) * inv_w, 0.0f), 63.0f)); };
                    for (int b = 0; b < nP; b += kWave) {
                        const int i = b + lane;
                        if (i < nP && F.pz[i] < take) atomicAdd(&F.hist[bin_of(F.pz[i])], 1u);
                        rejoin();
                    }
                    __syncthreads();
                    const int in_bin = int(F.hist[lane]);
                    int cum = in_bin;
#pragma unroll
                    for (int d = 1; d < kWave; d <<= 1) {
                        const int x = __shfl_up(cum, d);
                        if (lane >= d) cum += x;
                    }
                    // whole bins, as many as fit; where the first one with leaves is too many by itself, some
                    // of it (without progress in depth)
                    const uint64_t fit = wave_ballot(cum <= kFrontSorted), none = wave_ballot(cum == 0);
                    const bool partial = fit != ~0ull && (fit & ~none) == 0;
                    const int nbins = __popcll(partial ? none : fit) + (partial ? 1 : 0);
                    // a full pool keeps its nearest leaves alone, and this round ends in front of the others;
                    // where even those are too many, some of them are tested now
                    const float zcut = S0 + float(nbins) * wbin;
                    const bool cut = forced && !partial && zcut > B.zfrom * (1.0f + 4.0f * kFrontMargin) + 4.0f * B.pad;
                    const int total = __builtin_amdgcn_readlane(cum, nbins - 1);
                    const int nS = cut ? 0 : (total < kFrontSorted ? total : kFrontSorted);
                    F.hist[lane] = uint32_t(cum - in_bin);
                    __syncthreads();
                    int kept = 0;
                    float zleft = kInf;  // nearest leaf or node left for later
                    for (int b = 0; b < nP; b += kWave) {
                        const int i = b + lane;
                        const bool in = i < nP;
                        const float z = in ? F.pz[i] : kInf;
                        const int32_t js = in ? F.pr[i] : 0;
                        const int bin = bin_of(z);
                        bool sel = z < take && bin < nbins;
                        if (cut) {
                            sel = !sel;  // what does not stay
                        } else if (sel) {
                            const int at = int(atomicAdd(&F.hist[bin], 1u));
                            if (at < kFrontSorted) {
                                F.sz[at] = forced ? S0 : S0 + float(bin) * wbin;
                                F.sr[at] = js;
                            } else {
                                sel = false;
                            }
                        }
                        const uint64_t km = wave_ballot(in && !sel);
                        __syncthreads();
                        if (in && !sel) {
                            const int at = kept + int(lanes_below(km));
                            F.pz[at] = z;
                            F.pr[at] = js;
                            zleft = fminf(zleft, z);
                        }
                        kept += __popcll(km);
                        __syncthreads();
                    }
                    nP = kept;
                    if (cut) {
                        const double c = bound_key(fmaxf((zcut - ozr_of()) * (1.0f / dz_of()), 0.0f));
                        cap = c < cap ? c : cap;
                        B.zhi = uniform(fminf(B.zhi, zcut + kFrontMargin * zcut + B.pad));
                    }
                    // everything in front of `done` has been found
                    float done = forced || partial ? S0 : (nbins == kWave ? S1 : S0 + float(nbins) * wbin);
                    for (int b = 0; b < nN; b += kWave)
                        if (b + lane < nN) zleft = fminf(zleft, F.nz[b + lane]);
                    const float zmin = wave_min(zleft);
                    if (!forced) {
                        if (zmin > B.zhi) done = kInf;  // nothing is left, or nothing in reach
                        more = done < kInf;
                    }

                    // ---- test the leaves ray by ray, two at a time (their fetches and arithmetic overlap);
                    // behind the last ones, consume what the window settled
                    int32_t srv = 0, szv = 0;
                    int32_t reach = __float_as_int(B.zhi);  // depths are >= 0, so their bits order like integers
                    for (int i = 0;; i += 2) {
                        const bool end = i >= nS;
                        double ka = kNoHit, kb = kNoHit;
                        uint64_t ma = 0, mb = 0;
                        float oma = 1.0f, omb = 1.0f, ta = 0.0f, tb = 0.0f;
                        int32_t front = __float_as_int(done);
                        if (!end) {
                            const int ia = i & (kWave - 1);
                            if (ia == 0) {
                                const int at = i + lane < nS ? i + lane : nS - 1;
                                srv = F.sr[at];
                                szv = __float_as_int(F.sz[at]);
                            }
                            front = __builtin_amdgcn_readlane(szv, ia);
                            if (front > reach) continue;
                            ++tested;
                            const int64_t ja = __builtin_amdgcn_readlane(srv, ia), jb = __builtin_amdgcn_readlane(srv, ia + 1);
                            const float4 a0 = records[4 * ja], a1 = records[4 * ja + 1], a2 = records[4 * ja + 2],
                                         a3 = records[4 * ja + 3];
                            const float4 b0 = records[4 * jb], b1 = records[4 * jb + 1], b2 = records[4 * jb + 2],
                                         b3 = records[4 * jb + 3];
                            const uint32_t ga = uint32_t(gidx[ja]), gb = uint32_t(gidx[jb]);
                            HitGeom ha, hb2;
                            const float h2a = ellipsoid_h2(S.ray, a0, a1, a2, a3, ha);
                            const float h2b = ellipsoid_h2(S.ray, b0, b1, b2, b3, hb2);
                            asm volatile("" ::"s"(ga), "s"(gb));  // the index loads are issued with the records'
                            if (COUNT) {
                                cnt.leaf += i + 1 < nS ? 2 : 1;
                                cnt.lleaf += __popcll(on_mask) * (i + 1 < nS ? 2 : 1);
                            }
                            ma = wave_ballot(h2a <= P.Q) & on_mask;
                            mb = wave_ballot(h2b <= P.Q) & (i + 1 < nS ? on_mask : 0ull);
                            if ((ma | mb) == 0) continue;
                            ++useful;
                            ta = ellipsoid_t1(ha, a2, h2a, P.Q);
                            tb = ellipsoid_t1(hb2, b2, h2b, P.Q);
                            ka = hit_key(ta, ga);
                            kb = hit_key(tb, gb);
                            oma = 1.0f - a3.w * __expf(-0.5f * h2a);
                            omb = 1.0f - b3.w * __expf(-0.5f * h2b);
                            ma &= wave_ballot(ka < cap);
                            mb &= wave_ballot(kb < cap);
                            const uint64_t la = ma & ~wave_ballot(ka > S.last), lb = mb & ~wave_ballot(kb > S.last);
                            if (la | lb) {
                                // consumed in an earlier round (or in front of t_min), or found too late
                                if ((la & wave_ballot(ka > F.start[lane])) | (lb & wave_ballot(kb > F.start[lane]))) {
                                    redo = true;
                                    break;
                                }
                                ma &= ~la;
                                mb &= ~lb;
                            }
                            if ((ma | mb) == 0) continue;
                        }
                        if (end || ((ma | mb) & wave_ballot(hb.key[K - 2] != kNoHit))) {
                            // Consume the hits in front of `front` (their order is final): behind the last window
                            // all of them, else while many lanes have one or a lane with one has a full buffer
                            const int least = end ? (more ? 65 : 1) : kFrontDrain;
                            const float tf = (__int_as_float(front) - ozr_of()) * (1.0f / dz_of());
                            double key = hb.front();
                            int32_t js = inv[key != kNoHit ? hit_key_gid(key) : 0u];
                            for (;;) {
                                const uint64_t am = grp & wave_ballot(S.live) & wave_ballot(key != kNoHit) &
                                                    wave_ballot(hit_key_t(key) < tf) & wave_ballot(key < cap);
                                if (am == 0) break;
                                if (__popcll(am) < least && (am & wave_ballot(hb.key[K - 2] != kNoHit)) == 0) break;
                                if (COUNT) cnt.lcomp += __popcll(am);
                                const bool act = __builtin_amdgcn_inverse_ballot_w64(am);
                                const double key_s = key;
                                const int32_t js_s = js;
                                if (act) hb.pop_front();
                                rejoin();
                                key = hb.front();
                                js = inv[key != kNoHit ? hit_key_gid(key) : 0u];
                                consume<false, ROWS>(act, key_s, js_s, S, cold, records, ptr, P, zc, lists, LC, lane);
                            }
                            on_mask = grp & wave_ballot(S.live);
                            if (end || !on_mask) break;
                            ma &= on_mask;
                            mb &= on_mask;
                            if ((ma & ~wave_ballot(ka > S.last)) | (mb & ~wave_ballot(kb > S.last))) {
                                redo = true;
                                break;
                            }
                        }
                        if (COUNT) cnt.lbuf += __popcll(ma) + __popcll(mb);
                        const bool ca = __builtin_amdgcn_inverse_ballot_w64(ma), cb = __builtin_amdgcn_inverse_ballot_w64(mb);
                        if (ma) cap = min_bare(cap, hb.insert_out(ca ? ka : no_hit_here()));
                        if (mb) cap = min_bare(cap, hb.insert_out(cb ? kb : no_hit_here()));
                        // once the hits found so far bring T below eps1 whatever their order, none behind the
                        // farthest of them is wanted
                        Tv *= (ca ? oma : 1.0f) * (cb ? omb : 1.0f);
                        tv = fmaxf(tv, fmaxf(ca ? ta : 0.0f, cb ? tb : 0.0f));
                        const bool closed = Tv < closed_at;
                        if ((ma | mb) & wave_ballot(closed)) {
                            const double far = __longlong_as_double(__double_as_longlong(bound_key(tv)) + (1ll << 32));
                            cap = closed ? min_bare(cap, far) : cap;
                            const float zr = wave_max(__builtin_amdgcn_inverse_ballot_w64(on_mask)
                                                          ? __builtin_fmaf(hit_key_t(cap), dz_of(), ozr_of())
                                                          : -kInf);
                            reach = __float_as_int(zr + kFrontMargin * fabsf(zr) + B.pad);
                        }
                    }
                    if (redo || !on_mask) break;
                    if (tested > kFrontTested && 4 * useful < tested) {
                        leave = true;
                        break;
                    }
                    if (forced || !more) continue;

                    // ---- the next window starts at the nearest thing left
                    {
                        const bool on = __builtin_amdgcn_inverse_ballot_w64(on_mask);
                        const float dz = dz_of(), ozr = ozr_of();
                        const float zh = wave_max(on ? __builtin_fmaf(hit_key_t(cap), dz, ozr) : -kInf);
                        B.zhi = uniform(zh + kFrontMargin * fabsf(zh) + B.pad);
                        if (2 * __popcll(on_mask) <= n_on) {  // half of the rays have stopped: a tighter bundle
                            bundle_bounds(B, S.ray, on, ozr, dz);
                            n_on = __popcll(on_mask);
                        }
                    }
                    if (nS < 64) dS *= 2.0f;
                    if (nS > 144) dS *= 0.5f;
                    S0 = fmaxf(done, zmin);
                    S1 = S0 + fmaxf(dS, 1e-5f * S0 + 1e-20f);
                    int keep_n = 0;
                    for (int b = 0; b < nN; b += kWave) {
                        const int i = b + lane;
                        const bool in = i < nN;
                        const float z = in ? F.nz[i] : kInf;
                        const int32_t ref = in ? F.nr[i] : 0;
                        const uint64_t ma = wave_ballot(z < S1), mk = wave_ballot(in) & ~ma;
                        __syncthreads();
                        if (__builtin_amdgcn_inverse_ballot_w64(ma)) F.ar[nA + int(lanes_below(ma))] = ref;
                        if (__builtin_amdgcn_inverse_ballot_w64(mk)) {
                            const int at = keep_n + int(lanes_below(mk));
                            F.nz[at] = z;
                            F.nr[at] = ref;
                        }
                        nA += __popcll(ma);
                        keep_n += __popcll(mk);
                        __syncthreads();
                    }
                    nN = keep_n;
                }
                if (leave || redo) break;
                // a lane that lost nothing has consumed all its hits, every other live one those in front of
                // its cap
                if (__builtin_amdgcn_inverse_ballot_w64(on_mask) && !(cap < F.stop[lane])) S.live = false;
                rejoin();
                const uint64_t left = grp & wave_ballot(S.live);
                const float from = hit_key_t(cap);
                const uint64_t ahead = wave_ballot(S.last > F.start[lane]) | wave_ballot(from > F.from[lane]);
                const bool wide = P.pkt_shift == 6, sets = P.n_packets > P.packets_per_set;
                leave = left != 0 && (((left & ahead) == 0 && left == began) || ++rounds > kFrontRounds ||
                                      (rounds >= (wide ? kWideRounds : sets ? kSetsRounds : kSmallRounds) &&
                                       __popcll(left) >= (wide ? kWideLeft : sets ? kSetsLeft : kSmallLeft)));
                if (__builtin_amdgcn_inverse_ballot_w64(grp)) F.from[lane] = fmaxf(F.from[lane], from);
                rejoin();
            }
        }
        const LaneRay LR = lane_ray(P, ptr, pkt, lane);
        if (redo) {
            lane_reset<ROWS>(S, cold, LR.valid && P.n_gauss > 0 && LR.tmax > P.t_min, lane);
            LC = ListCursor{0, -1, 0, 0, LC.chunk, true};
        }
        if (wave_ballot(S.live)) {
            // with the stand-alone walk's buffer, its tail in the frontier's LDS
            static_assert(sizeof(FrontLds) >= sizeof(double) * kTailKeys * kWave, "room for the tail");
            using Buf = FwdBuf<48>::type;
            Buf wb;
            wb.ring = reinterpret_cast<double *>(&F);
            wb.lane = lane;
            __syncthreads();
            if (!walk_rounds<Buf, false, COUNT, false, ROWS>(S, cold, LR, zc, lists, LC, records, nodes, gidx, inv, ptr, P, wb, lane,
                                                       cnt))
                if (lane == 0) atomicOr(ptr.status, kStatusStack);
            __syncthreads();
        }
        write_rays<ROWS>(S, cold, LR, ptr.set[LR.si], ptr, LC, lists, lane);
        if (COUNT) {
            cnt.rows += uint64_t(LC.rows);
            cnt.slots += uint64_t(LC.slots);
        }
    }
    if (COUNT) add_counts(cnt, ptr, lane);
}

// ------------------------------------------------- adjoint by re-traversal

// The adjoint re-traverses each ray back to front: a round collects the K largest
// keys below the previous round's smallest (the first round: up to and including the
// last composited key the forward saved), keeping them in the hit buffer as negated
// keys so the same min/max network serves; nodes are culled against [K-th largest t,
// upper t] and the leader lane takes the child it leaves last first. The round's hits
// are then processed largest key first. Next to stored lists it serves the rays whose
// list is incomplete (the pool ran out).
template <int K, bool BRUTE, bool COUNT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(waves_for(K, true)))) void k_adjoint_trav(
    const float4 *__restrict__ records, const float4 *__restrict__ nodes, const int32_t *__restrict__ gidx,
    const int32_t *__restrict__ inv, const Ptrs ptr, const RenderParams P)
{
    constexpr bool kRev = true;
    if (P.overflow_only && uint32_t(ptr.pool.hdr[1]) == 0u) return;  // every list is complete
    const int lane = threadIdx.x;
    int64_t iter_pkt = 0;
    const int xcd = xcd_id();
    int qi = 0;
    uint64_t c_pkt = 0, c_node = 0, c_leaf = 0, c_round = 0, c_lleaf = 0, c_lbuf = 0, c_lcomp = 0, c_lchild = 0,
             c_group = 0;
    acc_clear(acc_table(), lane);
    for (;;) {
        const int64_t pkt = next_packet(P, ptr.queue, lane, xcd, qi, iter_pkt);
        if (pkt >= P.n_packets) break;
        if (COUNT) ++c_pkt;

        const LaneRay LR = lane_ray(P, ptr, pkt, lane);
        const RaySet &S = ptr.set[LR.si];
        const bool zc = S.zero_colour != 0;
        const bool valid = LR.valid;
        const int64_t ray_id = LR.id;
        const Ray ray = LR.ray;
        const float tmax = LR.tmax;
        const Slab sl = make_slab(ray);
        const int oct = wave_octant(sl, valid);

        LaneGrad Gd{0.0f, 0.0f, 0.0f};
        Back B{1.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0, -1};
        bool live = false;
        double hi = 0.0;  // keys of a round lie below it
        if (valid) {
            Gd.gr = S.grad[3 * ray_id];
            Gd.gg = S.grad[3 * ray_id + 1];
            Gd.gb = S.grad[3 * ray_id + 2];
            const uint4 ls = S.last[ray_id];
            B = back_init(S.fin[ray_id], ls, LR.bgr, LR.bgg, LR.bgb);
            live = ls.y != 0u && P.n_gauss > 0 && !(Gd.gr == 0.0f && Gd.gg == 0.0f && Gd.gb == 0.0f);
            if (P.overflow_only) {
                const int4 li = S.list[ray_id];
                live = live && li.y < li.x;
            }
            // the successor of the last composited key (next Gaussian index, same t)
            hi = __longlong_as_double((long long)(((uint64_t(ls.y) << 32) | ls.x) + 1ull));
        }
        bool overflow = false;

        while (wave_ballot(live)) {
            HitBuf<K> hb;  // negated keys, ascending: the largest key first
            hb.clear();
            if (COUNT) ++c_round;
            float t_lo = !live ? __builtin_nanf("") : P.t_min;  // rises to the K-th largest t
            const float t_hi_w = widen(hit_key_t(hi), sl.pad);

            const uint64_t live_now = wave_ballot(live);  // as in the forward's leaf step
            auto leaf = [&](int64_t j) {
                const int64_t js = __builtin_amdgcn_readfirstlane(int32_t(j));
                const float4 r0 = records[4 * js + 0], r1 = records[4 * js + 1], r2 = records[4 * js + 2],
                             r3 = records[4 * js + 3];
                const uint32_t gid = uint32_t(gidx[js]);
                HitGeom hg;
                const float h2 = ellipsoid_h2(ray, r0, r1, r2, r3, hg);
                // the index load is issued with the record's (its latency hides behind theirs)
                asm volatile("" ::"s"(gid));
                if (COUNT) {
                    ++c_leaf;
                    c_lleaf += __popcll(live_now);
                }
                const uint64_t hmask = wave_ballot(h2 <= P.Q) & live_now;
                if (!hmask) return;
                const float t1 = ellipsoid_t1(hg, r2, h2, P.Q);
                const double k = hit_key(t1, gid);
                const uint64_t cmask = hmask & wave_ballot(t1 >= P.t_min) & wave_ballot(t1 < tmax) & wave_ballot(k < hi) &
                                       wave_ballot(-k < hb.key[K - 1]);
                const bool cand = __builtin_amdgcn_inverse_ballot_w64(cmask);
                if (COUNT) c_lbuf += __popcll(cmask);
                if (cmask) {
                    hb.insert(cand ? -k : kNoHit);
                    if (hb.key[K - 1] != kNoHit) t_lo = fmaxf(P.t_min, hit_key_t(-hb.key[K - 1]));
                }
            };

            if (BRUTE) {
                for (int64_t j = 0; j < P.n_gauss; ++j) leaf(j);
            } else {
                RS_WALK_BVH()
            }
            if (overflow) {
                if (lane == 0) atomicOr(ptr.status, kStatusStack);
                live = false;
                break;
            }

            const double round_first = hb.key[K - 1];  // minus the round's smallest key (kNoHit: not full)
            bool more = true;
            for (int s = 0; s < K; ++s) {
                const double nk = hb.key[0];
                hb.pop_front();
                const bool act = more && live && nk != kNoHit;
                const uint64_t act_mask = wave_ballot(act);
                more = act_mask != 0;
                if (!more) break;
                if (COUNT) c_lcomp += __popcll(act_mask);
                const uint32_t gid = hit_key_gid(nk);
                HitData H;
                recompute_hit_at(act, gid, act ? inv[gid] : 0, ray, records, ptr.rgb, zc, P.Q, H);
                const float Tk = back_T(B, H.al);
                adjoint_hit<COUNT, true>(act, act_mask, gid, H, Tk, B, Gd, zc, ptr.gacc, lane, c_group);
                if (act) {
                    back_over(B, H.al, H.cr, H.cg, H.cb);
                    B.T = Tk;
                    ++B.done;
                }
            }
            // a lane whose buffer did not fill has reached its first hit
            if (live) {
                if (round_first == kNoHit)
                    live = false;
                else
                    hi = -round_first;
            }
        }
    }
    acc_flush<COUNT>(acc_table(), ptr.gacc, lane, c_group);
    if (COUNT && lane == 0 && c_pkt > 0) {
        atomicAdd(ptr.counters + 1, (unsigned long long)c_node);
        atomicAdd(ptr.counters + 2, (unsigned long long)c_leaf);
        atomicAdd(ptr.counters + 3, (unsigned long long)c_round);
        atomicAdd(ptr.counters + 4, (unsigned long long)c_lleaf);
        atomicAdd(ptr.counters + 5, (unsigned long long)c_lbuf);
        atomicAdd(ptr.counters + 6, (unsigned long long)c_lcomp);
        atomicAdd(ptr.counters + 7, (unsigned long long)c_lchild);
        atomicAdd(ptr.counters + 8, (unsigned long long)c_group);
        atomicAdd(ptr.counters + 13, (unsigned long long)c_pkt);
    }
}

// ------------------------------------------------- adjoint from stored lists

// The forward appended one row per compositing step of each packet; the adjoint
// walks the packet's rows from the last to the first, so every lane meets its
// own hits back to front (rows where it was idle hold kListIdle), and recomputes
// each hit with the forward's own per-hit arithmetic: no traversal and no hit
// buffer. The paper variant's second-phase hits (flagged, after the composited
// ones) only build the colour behind the last composited hit. Rays whose list is
// incomplete are left to the traversal adjoint.
// Bound by the gathers of records and the line atomics; the position lookup and the entries come one and two
// rows ahead (1M Gaussians, 1920x1080, forward's rows of this size: 2.75 ms, 2.94 with the lookup in line).
// Seven waves per SIMD: 2.75 ms; six 2.82, five 2.85.
constexpr int kListWaves = 7;
// Row cursor of the list adjoint (wave-uniform): `start` is where the row read last began,
// so the next row (back to front) ends there, or at the fill of an earlier chunk.
__device__ inline void row_seek(const int32_t *__restrict__ prev, const int32_t *__restrict__ fill, int32_t &chunk,
                                int32_t &start)
{
    // wave-uniform addresses, read through the constant address space (scalar loads)
    typedef const __attribute__((address_space(4))) int32_t *const_i32;
    while (start == 0 && chunk >= 0) {
        chunk = ((const_i32)prev)[chunk];
        start = chunk >= 0 ? ((const_i32)fill)[chunk] : 0;
    }
}

// Where the list adjoint stands: the row read last begins at slot `start` of `chunk`, `step` of its steps are left.
struct RowCursor {
    int32_t chunk, start, step;
    uint64_t mask;
};

// Moves to the step before, and returns whether there is one; `entry` is this lane's (kListIdle for a
// lane without one, or not live).
template <int ROWS>
__device__ inline bool step_back(const ListPool &pool, const int32_t *__restrict__ prev, const int32_t *__restrict__ fill,
                                 const uint32_t *__restrict__ slots, RowCursor &c, bool live, int lane, uint32_t &entry)
{
    entry = kListIdle;
    if (ROWS == 1 || c.step == 0) {
        row_seek(prev, fill, c.chunk, c.start);
        if (c.chunk < 0) return false;
        // the masks' address is wave-uniform: read it through the constant address space, so it is
        // a scalar load (the pool is only read by this kernel)
        typedef const __attribute__((address_space(4))) uint32_t *const_u32;
        const const_u32 mend = (const_u32)(slots + int64_t(c.chunk) * pool.chunk_slots + c.start - 2);
        c.mask = uint64_t(mend[0]) | (uint64_t(mend[1]) << 32);
        c.start -= __popcll(c.mask) + 2;
        c.step = ROWS == 1 ? 1 : row_steps(c.mask);
    }
    --c.step;
    const int sh = 16 * c.step;  // 0 where a row is one step
    const uint64_t m = c.mask >> sh;  // bits of later steps lie above the packet's lanes
    const uint32_t *row = slots + int64_t(c.chunk) * pool.chunk_slots + c.start + __popcll(c.mask & ((1ull << sh) - 1));
    const bool mine = ((m >> lane) & 1ull) != 0;
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(uint32_t(m >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(m), 0u));
    if (live && mine) entry = row[below];
    return true;
}

template <bool COUNT, int ROWS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kListWaves))) void k_adjoint_list(
    const float4 *__restrict__ records, const int32_t *__restrict__ inv, const Ptrs ptr, const RenderParams P)
{
    const int lane = threadIdx.x;
    int64_t iter_pkt = 0;
    const int xcd = xcd_id();
    int qi = 0;
    uint64_t c_pkt = 0, c_lcomp = 0, c_group = 0;
    // the pool is only read here
    const uint32_t *__restrict__ slots = ptr.pool.slots;
    const int32_t *__restrict__ prev = ptr.pool.prev;
    const int32_t *__restrict__ fill = ptr.pool.fill;
    for (;;) {
        const int64_t pkt = next_packet(P, ptr.queue, lane, xcd, qi, iter_pkt);
        if (pkt >= P.n_packets) break;
        if (COUNT) ++c_pkt;
        const LaneRay LR = lane_ray(P, ptr, pkt, lane);
        const RaySet &S = ptr.set[LR.si];
        const bool zc = S.zero_colour != 0;
        LaneGrad Gd{0.0f, 0.0f, 0.0f};
        Back B{1.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0, -1};
        int4 li = make_int4(0, 0, -1, 0);
        bool live = false;
        if (LR.valid) {
            li = S.list[LR.id];
            Gd.gr = S.grad[3 * LR.id];
            Gd.gg = S.grad[3 * LR.id + 1];
            Gd.gb = S.grad[3 * LR.id + 2];
            B = back_init(S.fin[LR.id], S.last[LR.id], LR.bgr, LR.bgg, LR.bgb);
            live = li.x > 0 && li.y == li.x && P.n_gauss > 0 && !(Gd.gr == 0.0f && Gd.gg == 0.0f && Gd.gb == 0.0f);
        }
        // the packet's last chunk (lane 0 always holds one of the packet's rays)
        int32_t chunk = __builtin_amdgcn_readfirstlane(li.z);
        if (!wave_ballot(live) || chunk < 0) continue;
        // Rows are walked from the last to the first: a row ends with its lane masks, so the
        // masks at the row's end give its start, which is the previous row's end. While a step is
        // processed, the next one's sorted positions and the one after that's entries are loaded, so
        // a step waits for its records alone.
        RowCursor rc{chunk, fill[chunk], 0, 0};
        uint32_t e1, e0 = kListIdle;
        int32_t js0 = 0;
        bool row1 = step_back<ROWS>(ptr.pool, prev, fill, slots, rc, live, lane, e1), row0 = true;
        while (row0) {
            const uint32_t cur = e0;
            const int32_t js = js0;
            e0 = e1;
            row0 = row1;
            js0 = inv[e0 != kListIdle ? e0 & ~kListSecond : 0u];  // idle lanes read Gaussian 0 (unused)
            e1 = kListIdle;
            if (row1) row1 = step_back<ROWS>(ptr.pool, prev, fill, slots, rc, live, lane, e1);
            const bool act = cur != kListIdle;
            if (!wave_ballot(act)) continue;
            const bool comp = act && cur < kListSecond;
            const uint32_t gid = act ? cur & ~kListSecond : 0u;
            HitData H;
            recompute_hit_at<true>(act, gid, js, LR.ray, records, ptr.rgb, zc, P.Q, H);
            const float Tk = back_T(B, H.al);
            const uint64_t comp_mask = wave_ballot(comp);
            if (COUNT) c_lcomp += __popcll(comp_mask);
            if (comp_mask)
                adjoint_hit<COUNT, false>(comp, comp_mask, gid, H, Tk, B, Gd, zc, ptr.gacc, lane, c_group);
            if (act) back_over(B, H.al, H.cr, H.cg, H.cb);
            if (comp) {
                B.T = Tk;
                ++B.done;
            }
        }
    }
    if (COUNT && lane == 0 && c_pkt > 0) {
        atomicAdd(ptr.counters + 9, (unsigned long long)c_pkt);
        atomicAdd(ptr.counters + 10, (unsigned long long)c_lcomp);
        atomicAdd(ptr.counters + 11, (unsigned long long)c_group);
    }
}

// ------------------------------------------------------------------- host

__global__ void k_zero_f32(float *p, int64_t n)
{
    int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    int64_t stride = int64_t(gridDim.x) * blockDim.x;
    for (; i < n; i += stride) p[i] = 0.0f;
}

// Accumulator (16 floats per Gaussian: body-frame mean 3, scale 3, angular 3,
// opacity 1, rgb 3, 3 unused) -> the caller's gradient arrays: dL/dm = -2 R acc_m
// and dL/dq = (2/|q|) E(q/|q|)^T acc_w (see grad_hit), with R^T from the
// Gaussian's record (the rotation the renders used).
__global__ __launch_bounds__(256) void k_scatter_grads(const float4 *__restrict__ gacc, const float4 *__restrict__ records,
                                                       const int32_t *__restrict__ inv, const float *__restrict__ quat,
                                                       int64_t n, float *d_mean, float *d_scale, float *d_quat,
                                                       float *d_opacity, float *d_rgb)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float4 a = gacc[4 * i], b = gacc[4 * i + 1], c = gacc[4 * i + 2], d = gacc[4 * i + 3];
    const float am0 = a.x, am1 = a.y, am2 = a.z, w0 = b.z, w1 = b.w, w2 = c.x;
    if (d_mean) {
        // R = (R^T)^T: dm_k = -2 sum_j RT_jk am_j
        const int32_t js = inv[i];
        const float4 r0 = records[4 * js], r1 = records[4 * js + 1], r2 = records[4 * js + 2];
        const float t00 = r0.x, t01 = r0.y, t02 = r0.z, t10 = r0.w, t11 = r1.x, t12 = r1.y, t20 = r1.z, t21 = r1.w,
                    t22 = r2.x;
        d_mean[3 * i] = -2.0f * (t00 * am0 + t10 * am1 + t20 * am2);
        d_mean[3 * i + 1] = -2.0f * (t01 * am0 + t11 * am1 + t21 * am2);
        d_mean[3 * i + 2] = -2.0f * (t02 * am0 + t12 * am1 + t22 * am2);
    }
    if (d_scale) {
        d_scale[3 * i] = a.w;
        d_scale[3 * i + 1] = b.x;
        d_scale[3 * i + 2] = b.y;
    }
    if (d_quat) {
        const float4 q = reinterpret_cast<const float4 *>(quat)[i];
        const float nq = sqrtf(q.x * q.x + q.y * q.y + q.z * q.z + q.w * q.w);
        const float in = 1.0f / nq, k = 2.0f * in;
        const float qw = q.x * in, vx = q.y * in, vy = q.z * in, vz = q.w * in;
        reinterpret_cast<float4 *>(d_quat)[i] =
            make_float4(-k * (vx * w0 + vy * w1 + vz * w2), k * (qw * w0 + (vy * w2 - vz * w1)),
                        k * (qw * w1 + (vz * w0 - vx * w2)), k * (qw * w2 + (vx * w1 - vy * w0)));
    }
    if (d_opacity) d_opacity[i] = c.y;
    if (d_rgb) {
        d_rgb[3 * i] = c.z;
        d_rgb[3 * i + 1] = c.w;
        d_rgb[3 * i + 2] = d.x;
    }
}

__global__ void k_zero_queue(uint32_t *q)
{
    if (threadIdx.x < kXcdQueues) q[threadIdx.x] = 0u;
}

__global__ void k_zero_pool_header(unsigned long long *h, unsigned long long second)
{
    if (threadIdx.x < 2) h[threadIdx.x] = threadIdx.x ? second : 0ull;
}

void reset_pool(const ListPool &pool, int pkt_shift, hipStream_t st)
{
    if (pool.hdr) k_zero_pool_header<<<1, 64, 0, st>>>(pool.hdr, (unsigned long long)pkt_shift << 32);
}

static void zero(float *p, int64_t n, hipStream_t st)
{
    if (!p || n <= 0) return;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    k_zero_f32<<<int(blocks), 256, 0, st>>>(p, n);
}

struct KernArgs {
    int grid;
    const float4 *records, *nodes;
    const int32_t *gidx, *inv;
};

// workgroups of a plain grid: one per packet, in whole deals (see next_packet)
static int plain_grid(int64_t n_packets)
{
    const int64_t deal = int64_t(kXcdQueues) * kXcdRun;
    return int((n_packets + deal - 1) / deal * deal);
}

template <int ROWS>
static void launch_adjoint_list(const KernArgs &a, const Ptrs &ptr, const RenderParams &P, hipStream_t st)
{
    if (P.count)
        k_adjoint_list<true, ROWS><<<a.grid, kWave, 0, st>>>(a.records, a.inv, ptr, P);
    else
        k_adjoint_list<false, ROWS><<<a.grid, kWave, 0, st>>>(a.records, a.inv, ptr, P);
}

template <int K, int ROWS>
static void launch_front(const KernArgs &a, const Ptrs &ptr, const RenderParams &P, hipStream_t st)
{
    if (P.count)
        k_render_front<K, true, ROWS><<<a.grid, kWave, 0, st>>>(a.records, a.nodes, a.gidx, a.inv, ptr, P);
    else
        k_render_front<K, false, ROWS><<<a.grid, kWave, 0, st>>>(a.records, a.nodes, a.gidx, a.inv, ptr, P);
}
template <int K>
static void launch_front(const KernArgs &a, const Ptrs &ptr, const RenderParams &P, hipStream_t st)
{
    if (P.lists && ptr.pool.chunk_slots != kChunkSlots)
        launch_front<K, kRowSteps>(a, ptr, P, st);
    else
        launch_front<K, 1>(a, ptr, P, st);
}

template <int K>
static void launch_k(Pass pass, const KernArgs &a, const Ptrs &ptr, const RenderParams &P, hipStream_t st)
{
    if (pass == Pass::Forward) {
        if (P.brute)
            k_render<K, true, false><<<a.grid, kWave, 0, st>>>(a.records, a.nodes, a.gidx, a.inv, ptr, P);
        else if (P.count)
            k_render<K, false, true><<<a.grid, kWave, 0, st>>>(a.records, a.nodes, a.gidx, a.inv, ptr, P);
        else
            k_render<K, false, false><<<a.grid, kWave, 0, st>>>(a.records, a.nodes, a.gidx, a.inv, ptr, P);
    } else {
        if (P.brute)
            k_adjoint_trav<K, true, false><<<a.grid, kWave, 0, st>>>(a.records, a.nodes, a.gidx, a.inv, ptr, P);
        else if (P.count)
            k_adjoint_trav<K, false, true><<<a.grid, kWave, 0, st>>>(a.records, a.nodes, a.gidx, a.inv, ptr, P);
        else
            k_adjoint_trav<K, false, false><<<a.grid, kWave, 0, st>>>(a.records, a.nodes, a.gidx, a.inv, ptr, P);
    }
}

void zero_gacc(const BvhDesc &D, hipStream_t st)
{
    Layout L = make_layout(D.n);
    zero(reinterpret_cast<float *>(D.ws + L.gacc), 16 * D.n, st);
}

void scatter_gacc(const BvhDesc &D, const float *quat, const rs_grads *grads, hipStream_t st)
{
    if (D.n <= 0) return;
    Layout L = make_layout(D.n);
    k_scatter_grads<<<int((D.n + 255) / 256), 256, 0, st>>>(
        reinterpret_cast<const float4 *>(D.ws + L.gacc), reinterpret_cast<const float4 *>(D.ws + L.records),
        reinterpret_cast<const int32_t *>(D.ws + L.inv), quat, D.n, grads->d_mean, grads->d_scale, grads->d_quat,
        grads->d_opacity, grads->d_rgb);
}

// One launch over up to kMaxSets ray sets sharing a layout (same count, same views).
int launch_sets(const BvhDesc &D, const rs_gaussians *g, const rs_params *p, int nsets, const SetDesc *sets,
                const ListRoom &room, Pass pass, hipStream_t st)
{
    Layout L = make_layout(D.n);
    char *ws = D.ws;
    WsHeader *h = reinterpret_cast<WsHeader *>(ws + L.header);
    const rs_rays *rays = sets[0].rays;

    RenderParams P{};
    P.n_rays = rays->n;
    P.n_gauss = D.n;
    P.root = D.root;
    P.stack_depth = p->stack_depth > 0 ? p->stack_depth : 64;
    P.Q = p->Q;
    P.eps1 = p->eps1;
    P.t_min = p->t_min;
    P.max_hits = p->max_hits;
    P.flags = p->flags;
    P.persistent = (p->flags & RS_PERSISTENT) ? 1 : 0;
    P.brute = (p->flags & RS_BRUTE_FORCE) ? 1 : 0;
    P.count = (p->flags & RS_COUNTERS) ? 1 : 0;
    P.front = pass == Pass::Forward && front_route(rays, nsets, p, D.n, room.units > 0);
    const int pkt_shift = P.front && room.units == 0 ? packet_shift_no_lists(rays, nsets, p, D.n)
                                                     : packet_shift(rays, nsets, p, D.n);
    const ListPool pool = list_pool_at(room, chunk_slots_of(pkt_shift));
    const int64_t packets = plan_packets(P, rays, pkt_shift == 6 ? tile_shift_of(p) : pkt_shift / 2, pkt_shift);
    P.packets_per_set = packets;
    P.n_packets = packets * nsets;
    P.strip_tiles = kStripTiles;
    P.lists = pool.chunks > 0 ? 1 : 0;
    P.overflow_only = (pass == Pass::AdjointTraverse && P.lists) ? 1 : 0;
    P.paper = (p->flags & RS_PAPER_GRADIENT) && P.lists ? 1 : 0;
    P.eps2 = p->eps2;
    P.chunk = (P.n_packets + kXcdQueues - 1) / kXcdQueues;

    Ptrs ptr{};
    ptr.rgb = g->rgb;
    for (int k = 0; k < kMaxSets; ++k) {
        const SetDesc &E = sets[k < nsets ? k : 0];
        RaySet &R = ptr.set[k];
        R.origin = E.rays->origin;
        R.dir = E.rays->dir;
        R.tmax = E.rays->t_max;
        R.bgray = E.rays->bg;
        R.grad = E.grad;
        R.out_rgb = E.out_rgb;
        R.fin = E.state.fin;
        R.last = E.state.last;
        R.list = E.state.list;
        for (int c = 0; c < 3; ++c) R.bg[c] = E.bg[c];
        R.zero_colour = E.zero_colour;
    }
    ptr.status = &h->status;
    ptr.queue = h->xq;
    ptr.counters = reinterpret_cast<unsigned long long *>(h->counters);
    ptr.gacc = reinterpret_cast<float *>(ws + L.gacc);
    ptr.pool = pool;

    if (pass == Pass::Forward && P.lists) reset_pool(pool, pkt_shift, st);
    if (P.n_packets > 0) {
        KernArgs a;
        const int kbuf = P.front ? front_keys(p->kbuf) : p->kbuf > 0 ? p->kbuf : 48;
        if (P.persistent) {
            k_zero_queue<<<1, 64, 0, st>>>(h->xq);
            int dev = 0, cus = 256;
            (void)hipGetDevice(&dev);
            (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
            // A workgroup for each wave that the CUs hold of this kernel; those beyond start late and find empty queues
            // (30k Gaussians, 400x300 with a mirror and shadows, forward: 1.25 ms; 1.35 at six waves per SIMD). The
            // list adjoint, which could hold seven, takes six: its waves' line atomics get in each other's way (500k,
            // 280x210 with a mirror 1.12 ms, 1.21 at seven; 4 x 1024x768 9.19 and 8.98). Brute force at 8 keys fits
            // one more than its target.
            const int per_simd = pass == Pass::AdjointList ? 6
                                 : P.front                 ? kFrontWaves
                                                           : waves_for(kbuf, pass != Pass::Forward) + P.brute;
            const int64_t waves = int64_t(cus) * 4 * per_simd;
            a.grid = int(waves < P.n_packets ? waves : P.n_packets);
        } else {
            a.grid = plain_grid(P.n_packets);
        }
        a.records = reinterpret_cast<const float4 *>(ws + L.records);
        a.nodes = reinterpret_cast<const float4 *>(ws + L.nodes);
        a.gidx = reinterpret_cast<const int32_t *>(ws + L.gidx);
        a.inv = reinterpret_cast<const int32_t *>(ws + L.inv);
        // the hit-buffer size never changes the result (same hits, same order, same arithmetic);
        // the default is the fastest measured size on MI355X
        if (pass == Pass::AdjointList) {
            if (ptr.pool.chunk_slots != kChunkSlots)
                launch_adjoint_list<kRowSteps>(a, ptr, P, st);
            else
                launch_adjoint_list<1>(a, ptr, P, st);
        } else if (P.front) {
            switch (kbuf) {
            case 16: launch_front<16>(a, ptr, P, st); break;
            case 24: launch_front<24>(a, ptr, P, st); break;
            default: launch_front<32>(a, ptr, P, st); break;
            }
        } else {
            switch (kbuf) {
            case 8: launch_k<8>(pass, a, ptr, P, st); break;
            case 16: launch_k<16>(pass, a, ptr, P, st); break;
            case 24: launch_k<24>(pass, a, ptr, P, st); break;
            case 32: launch_k<32>(pass, a, ptr, P, st); break;
            case 48: launch_k<48>(pass, a, ptr, P, st); break;
            default: return RS_ERR_INVALID_ARG;
            }
        }
    }
    return hipGetLastError() == hipSuccess ? RS_OK : RS_ERR_HIP;
}

int launch_render(const BvhDesc &D, const rs_gaussians *g, const rs_rays *rays, const rs_params *p,
                  float *out_rgb, void *state, const float *grad, const rs_grads *grads, hipStream_t st)
{
    const bool bwd = grad != nullptr;
    SetDesc S{};
    S.rays = rays;
    S.out_rgb = out_rgb;
    S.grad = grad;
    for (int c = 0; c < 3; ++c) S.bg[c] = p->bg[c];
    S.zero_colour = (p->flags & RS_ZERO_COLOUR) ? 1 : 0;
    const int32_t cap = p->hit_list;
    S.state = state_at(state, rays->n, cap);
    ListRoom pool{};
    if (state && cap > 0 && rays->n > 0) {
        const StateLayout sl = state_layout(rays->n, cap);
        pool = ListRoom{static_cast<char *>(state) + sl.pool, sl.chunks};
    }
    if (!bwd) return launch_sets(D, g, p, 1, &S, pool, Pass::Forward, st);
    int e;
    zero_gacc(D, st);
    if (pool.units > 0) {
        // stored lists first; the traversal adjoint then takes the rays whose list is
        // incomplete (it exits at once when the forward found the pool large enough).
        // The paper variant has no traversal form: its pool running out is an error.
        if ((e = launch_sets(D, g, p, 1, &S, pool, Pass::AdjointList, st))) return e;
        if (!(p->flags & RS_PAPER_GRADIENT))
            if ((e = launch_sets(D, g, p, 1, &S, pool, Pass::AdjointTraverse, st))) return e;
    } else {
        if ((e = launch_sets(D, g, p, 1, &S, pool, Pass::AdjointTraverse, st))) return e;
    }
    scatter_gacc(D, g->quat, grads, st);
    return hipGetLastError() == hipSuccess ? RS_OK : RS_ERR_HIP;
}

}  // namespace rs
