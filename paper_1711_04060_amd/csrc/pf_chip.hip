// pf_chip.hip -- on-chip Krylov kernel for gfx950.
//
// A BiCGSTAB run (Table 3, right Jacobi preconditioning, the scaled vectors
// and the two phases of pf_kernels.h) of a grid whose Krylov vectors fit the
// chip: 256 CUs hold 128 MB of registers and 40 MB of LDS, and the unknowns of
// a 129^3 grid take 86 MB.  The unknowns are cut into at most 256 boxes, one
// per workgroup and CU.  A thread owns a column of up to KZ nodes; r^ (s^ in
// its place), p^, v^, t^, x, the shadow and the classes of the node's
// neighbours stay in its registers for the whole run.  With 16 nodes a thread
// the registers are full: p^ is kept in LDS, and x in a piece of memory of the
// tile's own (it stays in the XCD's L2), updated while the tile waits for the
// others.  One launch runs every iteration until the stop test.
//
// Time per iteration against the two-kernel iteration (which reads and writes
// every vector each time, or, on small grids, waits for its launches and
// prologues), FP64 solves to 1e-12: 33^3 18.3 -> 7.7 us, 65^3 25.3 -> 9.2,
// 97^3 35.2 -> 12.6, 113^3 48.6 -> 21.7, 129^3 71.2 -> 24.3.
//
// What bounds it: an iteration has two grid-wide dependencies (alpha; omega
// and beta).  Each tile publishes its partial sums and the boundary values of
// the product it just formed (v^ or t^), and waits for those of the others:
// one exchange per dependency.  Every 8-byte word of an exchange holds 32 bits
// of data and the phase's tag, so the data say themselves that they have
// arrived: no flag follows them, and no fence writes back a cache (the buffer
// stores and loads have agent scope and go past the XCDs' own L2s).
// Neighbours' r^ and p^ at the halo nodes are not exchanged: every tile
// updates its copies with the recurrences, from the same operands.
//
// Buffers: phase n uses buffer n & 1.  A tile writes phase n + 2 after it has
// received every sum of phase n + 1, which each tile publishes after it has
// read phase n.  Tags are never used twice on the same buffers (the host
// counts them per grid), and the words that hold tags hold nothing else: every
// odd 32-bit word of the tagged block is a tag, in FP64 and FP32 and whatever
// the partition, and values without tags lie in a block of their own
// (chip_space).  In one block, a 16-plane run's plain values would stay behind
// where a later run looks for tags, and a plain FP32 value is a tag's bit
// pattern sooner or later.
//
// Every wait is bounded (spin polls).  A tile that gives up says so in the
// scalar block and leaves without writing x; the others, which wait for it in
// their turn, do the same, except where it gave up in the run's last phase: its
// own values are out by then, so others may receive everything, stop and write
// their part of x.  The caller therefore looks at gave_up before the stop
// state, takes x for one of mixed origin, and starts the two-kernel iteration
// from its true residual.  Tiles that do not give up decide from the same sums
// in the same order, so they leave in the same phase.
#include "pf_chip.h"

namespace pfk {

// Pauses (units of 64 cycles) before a tile's first poll and between polls:
// polls that come before the others' values compete with them for the fabric
// (all-gather of 5 sums among 256 tiles: 6967 cycles without, 2731 with 1024
// cycles of pause; among 64 tiles 4041 and 2336).
constexpr int CH_SLEEP0 = 12, CH_SLEEP = 2;      // tiles of up to 8 planes
constexpr int CH_SLEEPB0 = 32, CH_SLEEPB = 8;    // of 16

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr int SC1 = 16;   // agent scope of a buffer access

// Publish a value under a tag: {32 bits, tag} words.  SCOPE: SC1, or 0 where
// the reader shares the writer's L2.
template <int SCOPE>
__device__ __forceinline__ void xput(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, double v, unsigned tag)
{
    const u32x2 w = __builtin_bit_cast(u32x2, v);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{w.x, tag, w.y, tag}, b, at, base, SCOPE);
}
template <int SCOPE>
__device__ __forceinline__ void xput(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, float v, unsigned tag)
{
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{__builtin_bit_cast(unsigned, v), tag}, b, at, base, SCOPE);
}

// A published value as read: the words, whether they have arrived under the
// tag, and the value.  Loading and looking are apart so that every load of a
// poll is in flight before the first wait.
__device__ __forceinline__ void xload(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, u32x4 &w)
{
    w = __builtin_amdgcn_raw_buffer_load_b128(b, at, base, SC1);
}
__device__ __forceinline__ void xload(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, u32x2 &w)
{
    w = __builtin_amdgcn_raw_buffer_load_b64(b, at, base, SC1);
}
__device__ __forceinline__ bool xmiss(u32x4 w, unsigned tag) { return w.y != tag || w.w != tag; }
__device__ __forceinline__ bool xmiss(u32x2 w, unsigned tag) { return w.y != tag; }
__device__ __forceinline__ double xval(u32x4 w) { return __builtin_bit_cast(double, u32x2{w.x, w.z}); }
__device__ __forceinline__ float xval(u32x2 w) { return __builtin_bit_cast(float, w.x); }
// The same without a tag.
template <int SCOPE>
__device__ __forceinline__ void xput_plain(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, double v)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b, at, base, SCOPE);
}
template <int SCOPE>
__device__ __forceinline__ void xput_plain(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b, at, base, SCOPE);
}
__device__ __forceinline__ void xget_plain(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, double &v)
{
    v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, at, base, SC1));
}
__device__ __forceinline__ void xget_plain(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, float &v)
{
    v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, at, base, SC1));
}
// A tile's own memory (no other workgroup reads it).
__device__ __forceinline__ void xstore(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, double v)
{
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), b, at, base, 0);
}
__device__ __forceinline__ void xstore(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b, at, base, 0);
}
__device__ __forceinline__ void xfetch(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, double &v)
{
    v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b, at, base, 0));
}
__device__ __forceinline__ void xfetch(__amdgpu_buffer_rsrc_t b, unsigned at, unsigned base, float &v)
{
    v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, at, base, 0));
}
template <typename T> struct Word { using W = u32x4; };
template <> struct Word<float> { using W = u32x2; };

// Sum over the wave in lane 63 (DPP row shifts and broadcasts: a tenth of the
// latency of cross-lane permutes).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v)
{
    const u32x2 w = __builtin_bit_cast(u32x2, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0u, w.x, CTRL, ROWS, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0u, w.y, CTRL, ROWS, 0xf, true);
    return v + __builtin_bit_cast(double, u32x2{lo, hi});
}
template <int NQ>
__device__ __forceinline__ void wave_sums(double (&v)[NQ])
{
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = dpp_add<0x111, 0xf>(v[q]);   // row_shr 1, 2, 4, 8
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = dpp_add<0x112, 0xf>(v[q]);
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = dpp_add<0x114, 0xf>(v[q]);
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = dpp_add<0x118, 0xf>(v[q]);
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = dpp_add<0x142, 0xa>(v[q]);   // row_bcast 15, 31
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = dpp_add<0x143, 0xc>(v[q]);
}

__device__ __forceinline__ double uni(double x)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ float uni(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(unsigned, x)));
}

// First node of tile t of c along an axis of n unknowns from o (scalar: the
// division's result would stay in a vector register).
__device__ __forceinline__ int cut(int o, int n, int c, int t)
{
    return o + __builtin_amdgcn_readfirstlane(t * n / c);   // t <= 256 tiles, n <= 512 nodes each: t n <= 2^25
}

constexpr unsigned CH_DIR = 0x80000000u;

// x, in a way that keeps what is computed from it inside the iteration loop
// (hoisted out of it, every plane's table offsets would take registers for
// the whole run).
__device__ __forceinline__ unsigned here(unsigned x)
{
    asm volatile("" : "+v"(x));
    return x;
}
template <typename T>
__device__ __forceinline__ T here(T x)
{
    asm volatile("" : "+v"(x));
    return x;
}
__device__ __forceinline__ int here_s(int x)   // (a uniform value)
{
    asm volatile("" : "+s"(x));
    return x;
}

// LDS: KZ staged planes of the tile with its xy halo, the face table, the
// class shifts, p^ (KZ = 16).
template <typename T, int FORM, int KZ>
__global__ __launch_bounds__(CH_NT) void k_chip(const ChipSys<T> *__restrict__ table, const int *__restrict__ first,
                                                int nsys)
{
    constexpr int NT = CH_NT, LP = CH_LP, HS = chip_halo_slots(KZ), NW = NT / 64;
    constexpr int DUMMY = LP - 1;
    constexpr bool PAL = FORM != CHF_CEPS;
    constexpr bool BIG = KZ > 8;     // p^ in LDS, x in memory, classes packed (two-valued palettes only)
    constexpr int PG = KZ > 8 ? 2 : KZ > 4 ? 4 : 2;   // planes of a product handled together
    constexpr int UG = BIG && sizeof(T) == 4 ? 8 : 4;   // planes of a vector update handled together
    constexpr int RK = BIG ? 1 : KZ; // planes of the vectors that are in registers only when not BIG
    // Boundary values: under tags of their own on small tiles (one latency), as
    // plain values that the tile's tagged sums follow on larger ones (half the
    // bytes; the sums wait until the values are out)
    constexpr bool TAGGED = !BIG;
    constexpr unsigned EB = (TAGGED ? 2 : 1) * sizeof(T);   // bytes of an exchanged value
    extern __shared__ __align__(16) unsigned char smem[];
    T *const L = reinterpret_cast<T *>(smem);
    T *const ft = L + KZ * LP;
    T *const st = ft + FTAB;
    T *const PX = st + PAL_MAX;              // BIG: p^ of the own nodes
    __shared__ double stot[4][CH_NQ], bred[NW][CH_NQ];
    // (what only a failed poll needs is kept here: in registers it cost 2-4% of
    // an iteration)
    __shared__ int sfail, slimit;
    __shared__ __attribute__((address_space(1))) int *sgave;
    __shared__ unsigned snear;

    int si = 0, lb = blockIdx.x;
    if (nsys > 1) {
        int lo = 0, hi = nsys;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (first[mid] <= lb) lo = mid; else hi = mid;
        }
        si = __builtin_amdgcn_readfirstlane(lo);
        lb -= first[si];
    }
    const ChipSys<T> &S = table[si];
    const int nx = S.nx, ny = S.ny, nz = S.nz, P = S.P, G = S.ge.G;
    lb = xcd_remap(lb, G);   // an XCD's tiles lie together
    const int cx = S.ge.c[0], cy = S.ge.c[1], cz = S.ge.c[2];
    const int tz = __builtin_amdgcn_readfirstlane(lb / (cx * cy)), trow = lb - tz * cx * cy;
    const int ty = __builtin_amdgcn_readfirstlane(trow / cx), tx = trow - ty * cx;
    const int x0 = cut(S.ge.o[0], S.ge.n[0], cx, tx), y0 = cut(S.ge.o[1], S.ge.n[1], cy, ty),
              z0 = cut(S.ge.o[2], S.ge.n[2], cz, tz);
    const int bx = cut(S.ge.o[0], S.ge.n[0], cx, tx + 1) - x0, by = cut(S.ge.o[1], S.ge.n[1], cy, ty + 1) - y0,
              nk = cut(S.ge.o[2], S.ge.n[2], cz, tz + 1) - z0;
    const int W = bx + 2;
    const int tid = threadIdx.x;
    const bool act = tid < bx * by;
    const int j = act ? tid / bx : 0, i = act ? tid - j * bx : 0;
    const int gx = x0 + i, gy = y0 + j;
    const unsigned g0 = (unsigned)gx + (unsigned)nx * gy + (unsigned)P * z0;

    // neighbours in the staged planes (mirror ghosts on Neumann faces)
    const int a0 = (j + 1) * W + (i + 1);
    const int aw = act ? a0 : DUMMY;
    const int axm = gx == 0 ? a0 + 1 : a0 - 1, axp = gx == nx - 1 ? a0 - 1 : a0 + 1;
    const int aym = gy == 0 ? a0 + W : a0 - W, ayp = gy == ny - 1 ? a0 - W : a0 + W;
    const bool mlo = z0 == 0, mhi = z0 + nk == nz;   // the tile ends on a Neumann z face

    // exchange slots of the tile: its x, y and z faces (low, high)
    const int fx = S.ge.fx, fy = S.ge.fy, fz = S.ge.fz, fs = S.ge.fstride;
    const int bzlo = 2 * (fx + fy), bzhi = bzlo + fz;
    const bool zlo_in = act && tz > 0, zhi_in = act && tz < cz - 1;
    const int zoff = j * bx + i;
    // (absent neighbours: slot 0 is read and not used)
    const unsigned zsrc_lo = zlo_in ? (unsigned)((lb - cx * cy) * fs + bzhi + zoff) * EB : 0u;
    const unsigned zsrc_hi = zhi_in ? (unsigned)((lb + cx * cy) * fs + bzlo + zoff) * EB : 0u;
    // the boundary values this thread publishes: slot tid + u NT, staged at
    // pub[u] (DUMMY: a slot nobody reads)
    constexpr int FS = chip_face_slots(KZ);
    int pub[FS];
    unsigned side[FS];   // the face: -x +x -y +y -z +z
#pragma unroll
    for (int u = 0; u < FS; ++u) {
        int e = tid + u * NT, k = nk, q = 0;   // plane, index within the plane's staged cells
        side[u] = e < 2 * fx ? (e >= fx) : e < bzlo ? 2 + (e >= 2 * fx + fy) : 4 + (e >= bzhi);
        if (e < 2 * fx) {
            const bool up = e >= fx;
            if (up) e -= fx;
            if (up ? tx < cx - 1 : tx > 0) k = e / by;
            q = (e - k * by + 1) * W + (up ? bx : 1);
        } else if (e < bzlo) {
            const bool up = e >= 2 * fx + fy;
            e -= up ? 2 * fx + fy : 2 * fx;
            if (up ? ty < cy - 1 : ty > 0) k = e / bx;
            q = (up ? by : 1) * W + (e - k * bx + 1);
        } else if (e < fs) {
            const bool up = e >= bzhi;
            e -= up ? bzhi : bzlo;
            if (e < bx * by && (up ? tz < cz - 1 : tz > 0)) k = up ? nk - 1 : 0;
            q = (e / bx + 1) * W + (e % bx + 1);
        }
        pub[u] = k < nk ? k * LP + q : DUMMY;
    }

    if (tid == 0) {
        sfail = 0;
        slimit = S.spin;
        sgave = (__attribute__((address_space(1))) int *)&S.sc->gave_up;
    }
    for (int e = tid; e < KZ * LP; e += NT) L[e] = T(0);
    if constexpr (PAL) {
        if (tid < FTAB) ft[tid] = S.ftab[tid];
        if (FORM == CHF_CLASS && tid < PAL_MAX) st[tid] = S.stab[tid];
    }

    // own nodes
    T r[KZ], p[RK], v[KZ], t[KZ], xr[RK], sg[FORM == CHF_NODE ? KZ : 1];
    float rt[KZ];
    // per node: bits 0..3 own class, 4..27 the six neighbours', CH_DIR; BIG:
    // one byte, bit 0 own class, 1..6 the neighbours', 7 Dirichlet
    unsigned cls[BIG ? KZ / 4 : KZ];
    using GT = __attribute__((address_space(1))) T;
    GT *const gX = (GT *)S.x;
    // BIG: the tile's x, plane k of this thread at k NT + tid
    const auto xx = __builtin_amdgcn_make_buffer_rsrc(S.xtile + (BIG ? (size_t)lb * (KZ * NT) : 0), 0,
                                                      BIG ? (int)(KZ * NT * sizeof(T)) : 0, 0x00027000);
    const unsigned xat = tid * (unsigned)sizeof(T);
    constexpr unsigned XP = NT * sizeof(T);   // bytes of a plane
    const GT *const gS0 = (const GT *)S.s0;
    if constexpr (BIG) {
#pragma unroll
        for (int k = 0; k < KZ / 4; ++k) cls[k] = 0;
    }
    unsigned hom = 0, hcl = 0;   // planes (bits) on which the wave's nodes and neighbours all have class 0 / 1
#pragma unroll
    for (int k = 0; k < KZ; ++k) {
        r[k] = v[k] = t[k] = T(0);
        rt[k] = 0.0f;
        unsigned c = CH_DIR;
        if constexpr (FORM == CHF_NODE) sg[k] = T(0);
        T x = T(0);
        if (act && k < nk) {
            const unsigned g = g0 + (unsigned)P * k;
            r[k] = gS0[g];
            rt[k] = ((const __attribute__((address_space(1))) float *)S.rt)[g];
            if (!S.zero_x) x = gX[g];
            if constexpr (FORM == CHF_NODE) sg[k] = ((const GT *)S.sig)[g];
            if constexpr (PAL) {
                const auto *E = (const __attribute__((address_space(1))) uint8_t *)S.epsi;
                const int gz = z0 + k;
                const unsigned e = E[g];
                const unsigned n0 = E[gx == 0 ? g + 1 : g - 1] & 15u, n1 = E[gx == nx - 1 ? g - 1 : g + 1] & 15u;
                const unsigned n2 = E[gy == 0 ? g + nx : g - nx] & 15u, n3 = E[gy == ny - 1 ? g - nx : g + nx] & 15u;
                const unsigned n4 = E[gz == 0 ? g + P : g - P] & 15u, n5 = E[gz == nz - 1 ? g - P : g + P] & 15u;
                c = (e & 15u) | n0 << 4 | n1 << 8 | n2 << 12 | n3 << 16 | n4 << 20 | n5 << 24 |
                    ((e & 128u) ? CH_DIR : 0u);
            } else {
                c = (((const __attribute__((address_space(1))) uint8_t *)S.flags)[g] & S.dirbit) ? CH_DIR : 0u;
            }
        }
        if constexpr (!BIG) {
            xr[k] = x;
            p[k] = T(0);
            cls[k] = c;
        } else {
            PX[k * NT + tid] = T(0);
            xstore(xx, xat, k * XP, x);
            const unsigned m = (c & 1u) | (c >> 3 & 2u) | (c >> 6 & 4u) | (c >> 9 & 8u) | (c >> 12 & 16u) |
                               (c >> 15 & 32u) | (c >> 18 & 64u) | (c >> 24 & 128u);
            cls[k / 4] |= m << (8 * (k % 4));
        }
        if constexpr (PAL) {
            const bool fr = !(c & CH_DIR);
            const unsigned long long some = __ballot(fr);
            const unsigned cl = some ? __builtin_amdgcn_readlane(c, __ffsll((long long)some) - 1) & 15u : 0u;
            const bool odd = fr && c != cl * 0x1111111u;
            if (cl < 2 && !__any(odd)) {
                hom |= 1u << k;
                hcl |= cl << k;
            }
        }
    }
    hom = __builtin_amdgcn_readfirstlane(hom);
    hcl = __builtin_amdgcn_readfirstlane(hcl);

    // halo nodes: xy halo (HS slots per thread) and the two z neighbours
    T hr[HS], hp[HS], hv[HS];
    unsigned hsrc[HS];
    int hl[HS];
    bool hin[HS];
    const int h1 = by * nk, h2 = 2 * h1, h3 = h2 + bx * nk, h4 = h3 + bx * nk;
#pragma unroll
    for (int u = 0; u < HS; ++u) {
        const int h = tid + u * NT;
        hr[u] = hp[u] = hv[u] = T(0);
        hsrc[u] = 0u;
        hin[u] = false;
        hl[u] = DUMMY;
        if (h < h4) {
            int hi_, hj, hk, src = -1;
            if (h < h2) {
                const bool up = h >= h1;
                const int e = up ? h - h1 : h;
                hk = e / by;
                hj = e - hk * by;
                hi_ = up ? bx : -1;
                if (up ? tx < cx - 1 : tx > 0) src = (up ? lb + 1 : lb - 1) * fs + (up ? 0 : fx) + e;
            } else {
                const bool up = h >= h3;
                const int e = up ? h - h3 : h - h2;
                hk = e / bx;
                hi_ = e - hk * bx;
                hj = up ? by : -1;
                if (up ? ty < cy - 1 : ty > 0) src = (up ? lb + cx : lb - cx) * fs + 2 * fx + (up ? 0 : fy) + e;
            }
            if (src >= 0) {
                hsrc[u] = (unsigned)src * EB;
                hin[u] = true;
                hl[u] = hk * LP + (hj + 1) * W + hi_ + 1;
                hr[u] = gS0[(unsigned)(x0 + hi_) + (unsigned)nx * (y0 + hj) + (unsigned)P * (z0 + hk)];
            }
        }
    }
    T zr[2] = {T(0), T(0)}, zp[2] = {T(0), T(0)}, zv[2] = {T(0), T(0)};
    if (zlo_in) zr[0] = gS0[g0 - P];
    if (zhi_in) zr[1] = gS0[g0 + (unsigned)P * nk];
    __syncthreads();

    // face coefficient, diagonal and its inverse of homogeneous planes
    T hc0 = T(0), hc1 = T(0), hD0 = T(0), hD1 = T(0), hi0 = T(0), hi1 = T(0);
    if constexpr (PAL) {
        hc0 = uni(ft[0]);
        hc1 = uni(ft[PAL_MAX + 1]);
        hD0 = ((hc0 + hc0) + (hc0 + hc0)) + (hc0 + hc0);
        hD1 = ((hc1 + hc1) + (hc1 + hc1)) + (hc1 + hc1);
        if constexpr (FORM == CHF_CLASS) {
            hD0 += st[0];
            hD1 += st[1];
        }
        hi0 = uni((T)rcp_pos(hD0));
        hi1 = uni((T)rcp_pos(hD1));
        hD0 = uni(hD0);
        hD1 = uni(hD1);
    }
    const T ceps = S.ceps, cdiag = S.cdiag, cidiag = S.cidiag;

    // Cell a of staged plane k.  An address beyond the 16 bits of an LDS
    // instruction's offset is computed here (outside of the iteration loop it
    // would take a register, which the 16-plane instances reload from memory).
    auto cell = [&](const int k, const int a) -> T & {
        return L[((k + 1) * LP * (int)sizeof(T) > 0xffff ? here(a) : a) + k * LP];
    };

    // A q (aq) and D^-1 A q (hat) at planes k0 .. k0 + PG - 1 of the own column,
    // with the diagonal D; q in registers, its z halo in zl, zh.  The LDS reads
    // of all planes go out first.  A wave whose nodes and neighbours are all of
    // one class on all of these planes (most are) needs no coefficient lookup.
    // Q(k): q at plane k.
    auto product = [&](const int k0, auto Q, const T zl, const T zh, T(&aq)[PG], T(&D)[PG], T(&hat)[KZ]) {
        T l[PG][4], zd[PG], zu[PG], sum[PG], iD[PG], qc[PG + 2];
#pragma unroll
        for (int e = 0; e < PG; ++e) {
            l[e][0] = cell(k0 + e, axm);
            l[e][1] = cell(k0 + e, axp);
            l[e][2] = cell(k0 + e, aym);
            l[e][3] = cell(k0 + e, ayp);
        }
#pragma unroll
        for (int e = 0; e < PG + 2; ++e) {   // planes k0 - 1 .. k0 + PG
            const int k = k0 + e - 1;
            qc[e] = k < 0 ? zl : k < KZ ? Q(k < 0 ? 0 : k < KZ ? k : 0) : zh;
        }
#pragma unroll
        for (int e = 0; e < PG; ++e) {
            const int k = k0 + e;
            const bool last = k == nk - 1;
            zd[e] = qc[e];
            zu[e] = last ? zh : qc[e + 2];
            if (last && mhi) zu[e] = zd[e];
            if (k == 0 && mlo) zd[e] = zu[e];
        }
        if constexpr (FORM == CHF_CEPS) {
#pragma unroll
            for (int e = 0; e < PG; ++e) {
                sum[e] = ceps * (l[e][0] + l[e][1] + l[e][2] + l[e][3] + zu[e] + zd[e]);
                D[e] = cdiag;
                iD[e] = cidiag;
            }
        } else if ((((unsigned)here_s(hom) >> k0) & ((1u << PG) - 1)) == (1u << PG) - 1) {
            const unsigned hk = (unsigned)here_s(hcl) >> k0;
#pragma unroll
            for (int e = 0; e < PG; ++e) {
                const bool c1 = (hk >> e) & 1u;
                const T c = c1 ? hc1 : hc0;
                sum[e] = c * l[e][0] + c * l[e][1] + c * l[e][2] + c * l[e][3] + c * zd[e] + c * zu[e];
                D[e] = c1 ? hD1 : hD0;
                iD[e] = c1 ? hi1 : hi0;
                if constexpr (FORM == CHF_NODE) {
                    D[e] += here(sg[k0 + e]);
                    iD[e] = rcp_pos(D[e]);
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < PG; ++e) {
                constexpr unsigned B = BIG ? 1 : 4, M = BIG ? 1 : 15;
                const unsigned m = BIG ? here(cls[(k0 + e) / 4]) >> (8 * ((k0 + e) % 4)) : here(cls[BIG ? 0 : k0 + e]);
                const T *row = ft + (m & M) * PAL_MAX;
                const T c0 = row[(m >> B) & M], c1 = row[(m >> 2 * B) & M], c2 = row[(m >> 3 * B) & M];
                const T c3 = row[(m >> 4 * B) & M], c4 = row[(m >> 5 * B) & M], c5 = row[(m >> 6 * B) & M];
                sum[e] = c0 * l[e][0] + c1 * l[e][1] + c2 * l[e][2] + c3 * l[e][3] + c4 * zd[e] + c5 * zu[e];
                D[e] = ((c0 + c1) + (c2 + c3)) + (c4 + c5);
                if constexpr (FORM == CHF_NODE) D[e] += here(sg[k0 + e]);
                if constexpr (FORM == CHF_CLASS) D[e] += st[m & M];
                iD[e] = rcp_pos(D[e]);
            }
        }
#pragma unroll
        for (int e = 0; e < PG; ++e) {
            const unsigned m = here(cls[BIG ? (k0 + e) / 4 : k0 + e]);
            const bool dir = BIG ? (m >> (8 * ((k0 + e) % 4) + 7)) & 1u : (int)m < 0;
            aq[e] = dir ? T(0) : D[e] * qc[e + 1] - sum[e];
            hat[k0 + e] = aq[e] * iD[e];
        }
    };

    // halo values into the staged planes
    auto stage_halo = [&](const T(&h)[HS]) {
#pragma unroll
        for (int u = 0; u < HS; ++u) L[hl[u]] = h[u];
    };

    // exchange: two buffers of face values, then two of sums
    const unsigned fbuf = (unsigned)(G * fs) * EB;
    const auto xf = __builtin_amdgcn_make_buffer_rsrc(S.face, 0, (int)(2 * fbuf), 0x00027000);
    // sums: two buffers of the tiles' (a row of GR words per group and
    // quantity; or all tiles as one group), two of the groups', XCD ids
    constexpr unsigned GR = CH_GMAX / 8, SB1 = 8 * CH_NQ * GR * 16, SB2 = CH_NQ * 8 * 16;
    const auto xs = __builtin_amdgcn_make_buffer_rsrc(S.sums, 0, (int)(2 * SB1), 0x00027000);
    const auto xg = __builtin_amdgcn_make_buffer_rsrc((char *)S.sums + 2 * SB1, 0, (int)(2 * SB2), 0x00027000);
    const auto xi = __builtin_amdgcn_make_buffer_rsrc((char *)S.sums + 2 * (SB1 + SB2), 0, 8 * CH_GMAX, 0x00027000);
    // Of more than 128 tiles, each group (the tiles xcd_remap gives one XCD)
    // adds up first: its first tile takes the members' sums and publishes
    // theirs, and every tile takes the eight groups'.  (All tiles reading all
    // sums moved 3.7 MB an exchange and poll at 216 tiles: 14.0 us an iteration
    // at 97^3, 12.3 this way; at 49^3 with 108 tiles it is 8.3 against 9.6,
    // and with 16 planes a tile, where phases are long, 19.9 against 20.9 at
    // 113^3.)
    const bool two = !BIG && G > 128;
    const int gper = G / 8, grem = G % 8, gcut = grem * (gper + 1);
    const int grp = !two ? 0 : __builtin_amdgcn_readfirstlane(lb < gcut ? lb / (gper + 1) : grem + (lb - gcut) / gper);
    const int gat = !two ? 0 : grp * gper + (grp < grem ? grp : grem);    // first tile of the group
    const int gsz = !two ? G : gper + (grp < grem ? 1 : 0);
    const unsigned grow = two ? GR : (unsigned)G;                                // words of a row
    const unsigned gbase = (unsigned)grp * (CH_NQ * GR) * 16u;
    const unsigned tag0 = S.tag0;
    // the neighbours on this XCD (bit per face): their values go through its
    // L2 only (nearby tiles are, where the dispatcher deals the workgroups to
    // the XCDs in turn; the ids are the hardware's own)
    const unsigned xcc = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15u;   // HW_REG_XCC_ID
    auto give_up = [&]() {
        sfail = 1;
        __hip_atomic_store(sgave, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    unsigned near = 0;
    if (tid < 64) {
        if (tid == 0) __builtin_amdgcn_raw_buffer_store_b64(u32x2{xcc, tag0}, xi, (unsigned)lb * 8u, 0, SC1);
        const int dn[6] = {tx > 0 ? -1 : 0, tx < cx - 1 ? 1 : 0, ty > 0 ? -cx : 0, ty < cy - 1 ? cx : 0,
                           tz > 0 ? -cx * cy : 0, tz < cz - 1 ? cx * cy : 0};
        // lanes 0..5: the face neighbours; from 8 on: the group's tiles
        int d = two && tid >= 8 && tid - 8 < gsz ? gat + tid - 8 - lb : 0;
#pragma unroll
        for (int f = 0; f < 6; ++f) d = tid == f ? dn[f] : d;
        u32x2 w;
        for (int spin = 0;; ++spin) {
            w = __builtin_amdgcn_raw_buffer_load_b64(xi, (unsigned)(lb + d) * 8u, 0, SC1);
            if (!__any(w.y != tag0)) break;
            if (spin >= slimit) {
                give_up();
                break;
            }
            __builtin_amdgcn_s_sleep(CH_SLEEP);
            asm volatile("" ::: "memory");
        }
        const unsigned long long same = __ballot(w.x == xcc);
        near = (unsigned)(same & 63u) | ((same >> 8) == (~0ull >> 8) && two ? 64u : 0u);   // bit 6: the whole group
        if (tid == 0) snear = near;
    }
    __syncthreads();
    if (sfail) return;
    near = snear;
    unsigned local = 0;   // bit u: slot u's reader is near
#pragma unroll
    for (int u = 0; u < FS; ++u) local |= ((near >> side[u]) & 1u) << u;
    // phase n: the tile's sums, and the boundary values of val, which takes
    // the staged planes' own cells (whole lines per wave go out)
    auto publish = [&](const int n, const T(&val)[KZ], auto &acc) {
        constexpr int NQ = sizeof(acc) / sizeof(double);
        __syncthreads();   // the staged planes have been read
#pragma unroll
        for (int k = 0; k < KZ; ++k)
            if (k / UG * UG < nk) cell(k, aw) = val[k];
        wave_sums<NQ>(acc);
        if ((tid & 63) == 63) {
#pragma unroll
            for (int q = 0; q < NQ; ++q) bred[tid >> 6][q] = acc[q];
        }
        __syncthreads();
        const unsigned base = (n & 1) * fbuf + (unsigned)(lb * fs) * EB;
        if constexpr (!TAGGED) {
#pragma unroll
            for (int u = 0; u < FS; ++u)
                if (pub[u] != DUMMY) {
                    const unsigned at = (unsigned)(tid + u * NT) * EB;
                    xput_plain<SC1>(xf, at, base, L[pub[u]]);
                }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's values are out
            __syncthreads();                                   // every wave's
        }
        if (tid < NQ) {
            double s = bred[0][tid];
#pragma unroll
            for (int w = 1; w < NW; ++w) s += bred[w][tid];
            const unsigned at = (unsigned)((BIG ? here(tid) : tid) * grow + (lb - gat)) * 16u, sb = (n & 1) * SB1 + gbase;
            if (!BIG && (near & 64u)) xput<0>(xs, at, sb, s, tag0 + n);
            else xput<SC1>(xs, at, sb, s, tag0 + n);
        }
        if constexpr (TAGGED) {
#pragma unroll
            for (int u = 0; u < FS; ++u)
                if (pub[u] != DUMMY) {
                    const unsigned at = (unsigned)(tid + u * NT) * EB;
                    if ((local >> u) & 1u) xput<0>(xf, at, base, L[pub[u]], tag0 + n);
                    else xput<SC1>(xf, at, base, L[pub[u]], tag0 + n);
                }
        }
    };
    // wait for phase n: halo values into h, z, the grid's sums into tot;
    // false: gave up
    auto receive = [&](const int n, T(&h)[HS], T(&z)[2], auto &tot) -> bool {
        constexpr int NQ = sizeof(tot) / sizeof(double);
        const unsigned base = (n & 1) * fbuf, sb = (n & 1) * SB1 + gbase, tag = tag0 + n;
        using W = typename Word<T>::W;
        double s[NQ];
        const bool summers = tid < 64 || (!two && (tid & ~63) < G);   // uniform in a wave
        // the sums of this tile's group into s (lane: tile), once
        const bool summer = tid < gsz;   // (two: of the first wave only)
        const unsigned sat = (summer ? (unsigned)tid : 0u) * 16u;
        auto group_sums = [&]() -> bool {
            u32x4 sw[NQ];
            bool miss = false;
#pragma unroll
            for (int q = 0; q < NQ; ++q) xload(xs, sat, sb + (unsigned)q * grow * 16u, sw[q]);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                miss |= summer && xmiss(sw[q], tag);
                s[q] = summer ? xval(sw[q]) : 0.0;
            }
            return miss;
        };
        if (two && tid < 64 && lb == gat) {
            for (int spin = 0;; ++spin) {
                if (!__any(group_sums())) break;
                if (spin >= slimit) {
                    give_up();
                    break;
                }
                asm volatile("" ::: "memory");   // every poll reads again
            }
            wave_sums<NQ>(s);
            if (tid == 63 && !sfail) {
#pragma unroll
                for (int q = 0; q < NQ; ++q) xput<SC1>(xg, (unsigned)(q * 8 + grp) * 16u, (n & 1) * SB2, s[q], tag);
            }
        }
        __builtin_amdgcn_s_sleep(BIG ? CH_SLEEPB0 : CH_SLEEP0);
        double gs = 0.0;   // two: lane 8 q + g holds quantity q of group g
        for (int spin = 0; TAGGED || summers; ++spin) {
            W hw[HS], zw[2];
            bool miss = false;
            if constexpr (TAGGED) {
#pragma unroll
                for (int u = 0; u < HS; ++u) xload(xf, hsrc[u], base, hw[u]);
                xload(xf, zsrc_lo, base, zw[0]);
                xload(xf, zsrc_hi, base, zw[1]);
            }
            if (summers) {
                if (two) {
                    u32x4 w;
                    const bool in = tid < 8 * NQ;
                    xload(xg, (in ? (unsigned)tid : 0u) * 16u, (n & 1) * SB2, w);
                    miss = in && xmiss(w, tag);
                    gs = in ? xval(w) : 0.0;
                } else {
                    miss = group_sums();
                }
            }
            if constexpr (TAGGED) {
#pragma unroll
                for (int u = 0; u < HS; ++u) {
                    miss |= hin[u] && xmiss(hw[u], tag);
                    h[u] = hin[u] ? xval(hw[u]) : T(0);
                }
                miss |= (zlo_in && xmiss(zw[0], tag)) || (zhi_in && xmiss(zw[1], tag));
                z[0] = zlo_in ? xval(zw[0]) : T(0);
                z[1] = zhi_in ? xval(zw[1]) : T(0);
            }
            if (!__any(miss)) break;
            if (spin >= slimit) {
                give_up();
                break;
            }
            __builtin_amdgcn_s_sleep(BIG ? CH_SLEEPB : CH_SLEEP);
            asm volatile("" ::: "memory");   // every poll reads again
        }
        if (summers) {
            if (two) {
                gs = dpp_add<0x111, 0xf>(gs);   // over the eight lanes of a quantity
                gs = dpp_add<0x112, 0xf>(gs);
                gs = dpp_add<0x114, 0xf>(gs);
                if ((tid & 7) == 7 && tid < 8 * NQ) stot[0][tid >> 3] = gs;
            } else {
                wave_sums<NQ>(s);
                if ((tid & 63) == 63) {
#pragma unroll
                    for (int q = 0; q < NQ; ++q) stot[tid >> 6][q] = s[q];
                }
            }
        }
        __syncthreads();
        if constexpr (!TAGGED) {   // every tile's sums are here, so its values are out
#pragma unroll
            for (int u = 0; u < HS; ++u) xget_plain(xf, hsrc[u], base, h[u]);
            xget_plain(xf, zsrc_lo, base, z[0]);
            xget_plain(xf, zsrc_hi, base, z[1]);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            double a = stot[0][q];
            if (!two)
                for (int w = 1; w < (G + 63) >> 6; ++w) a += stot[w][q];
            tot[q] = uni(a);
        }
        if constexpr (!TAGGED) {
#pragma unroll
            for (int u = 0; u < HS; ++u) h[u] = hin[u] ? h[u] : T(0);
            z[0] = zlo_in ? z[0] : T(0);
            z[1] = zhi_in ? z[1] : T(0);
        }
        return sfail == 0;
    };

    // BIG: x += the change in t.  The tile's x lies together in memory, so that
    // an XCD's tiles keep theirs in its L2 (in the grid's own layout the lines
    // that tiles share did not stay there: 14000 cycles at 129^3).
    auto update_x = [&]() {
        if constexpr (BIG) {
#pragma unroll
            for (int k0 = 0; k0 < KZ; k0 += 8) {
                if (k0 < nk) {
                    T x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) xfetch(xx, xat, (k0 + e) * XP, x[e]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) xstore(xx, xat, (k0 + e) * XP, x[e] + t[k0 + e]);
                }
            }
        }
    };

    // scalars of the run (Scalars slot 1: the previous iteration's)
    Scalars sc = S.init;
    sc.rho[1] = sc.rho[0];
    int iter = sc.iter[0];
    double rho = sc.rho[0], rr = sc.rr;
    int stop = ST_RUN;
    bool fresh = true, upx = false;   // upx: leave with a change of x in t
    int ph = 0;
    for (;;) {
        // ---- step A: finish the previous iteration, p^, v^ = D^-1 A p^
        T be = T(0), om = T(0);
        if (!fresh) {
            double tot[5];
            T ht[HS], zt[2] = {T(0), T(0)};
#pragma unroll
            for (int u = 0; u < HS; ++u) ht[u] = T(0);
            if (!receive(ph - 1, ht, zt, tot)) return;
            const FinB f = fin_b(&sc, tot, 0);
            if (f.update) {
                iter = f.iter;
                rho = f.rho;
                rr = f.rr;
            }
            stop = f.stop;
            if (!f.update) break;
            om = (T)uni(f.omega);
            be = (T)uni(f.beta);
            const T al = (T)uni(f.alpha);
#pragma unroll
            for (int k0 = 0; k0 < KZ; k0 += UG) {
                if (k0 < nk) {
                    T po[UG];
#pragma unroll
                    for (int e = 0; e < UG; ++e) po[e] = BIG ? PX[(k0 + e) * NT + tid] : p[BIG ? 0 : k0 + e];
#pragma unroll
                    for (int e = 0; e < UG; ++e) {
                        const int k = k0 + e;
                        const T s = r[k];
                        r[k] = s - om * t[k];
                        const T pn = r[k] + be * (po[e] - om * v[k]);
                        if constexpr (BIG) {
                            // the change of x takes t^'s registers until the shadow of this step
                            t[k] = al * po[e] + om * s;
                            PX[k * NT + tid] = pn;
                        } else {
                            xr[k] = xr[k] + al * po[e] + om * s;
                            p[k] = pn;
                        }
                        cell(k, aw) = pn;
                    }
                }
            }
            if (stop != ST_RUN) {
                upx = true;
                break;
            }
#pragma unroll
            for (int u = 0; u < HS; ++u) hr[u] = hr[u] - om * ht[u];
            zr[0] = zr[0] - om * zt[0];
            zr[1] = zr[1] - om * zt[1];
        }
        if (fresh) {
#pragma unroll
            for (int k = 0; k < KZ; ++k) {
                if constexpr (BIG) PX[k * NT + tid] = r[k];
                else p[k] = r[k];
                cell(k, aw) = r[k];
            }
        }
#pragma unroll
        for (int u = 0; u < HS; ++u) hp[u] = hr[u] + be * (hp[u] - om * hv[u]);
        zp[0] = zr[0] + be * (zp[0] - om * zv[0]);
        zp[1] = zr[1] + be * (zp[1] - om * zv[1]);
        stage_halo(hp);
        __syncthreads();
        {
            double acc[2] = {0.0, 0.0};
#pragma unroll
            for (int k0 = 0; k0 < KZ; k0 += PG) {
                if (k0 < nk) {
                    T a[PG], D[PG];
                    product(k0, [&](int k) -> T { return BIG ? PX[k * NT + tid] : p[BIG ? 0 : k]; }, zp[0], zp[1], a, D, v);
#pragma unroll
                    for (int e = 0; e < PG; ++e) {
                        const double rk = (double)D[e] * (double)r[k0 + e];
                        acc[0] += (double)rt[k0 + e] * (double)a[e];
                        acc[1] += rk * rk;
                    }
                }
                if constexpr (KZ > 8) __builtin_amdgcn_sched_barrier(0);
            }
            publish(ph, v, acc);
        }
        if constexpr (BIG) {
            if (!fresh) update_x();
        }
        ++ph;
        // ---- step B: s^ = r^ - alpha v^, t^ = D^-1 A s^
        double tot2[2];
        if (!receive(ph - 1, hv, zv, tot2)) return;
        rr = tot2[1];
        double alpha = 0.0;
        if (!finite(tot2[0]) || !finite(rr)) stop = ST_NONFINITE;
        else if (rr <= sc.tol2) stop = ST_CONV;
        else if (iter >= sc.maxit) stop = ST_MAXIT;
        else if (tot2[0] == 0.0) stop = ST_RESTART;
        else alpha = uni(rho / tot2[0]);
        if (stop != ST_RUN) break;
        const T al = (T)alpha;
#pragma unroll
        for (int k = 0; k < KZ; ++k) {
            if (k / UG * UG < nk) {
                r[k] = r[k] - al * v[k];
                cell(k, aw) = r[k];
            }
        }
#pragma unroll
        for (int u = 0; u < HS; ++u) hr[u] = hr[u] - al * hv[u];
        zr[0] = zr[0] - al * zv[0];
        zr[1] = zr[1] - al * zv[1];
        stage_halo(hr);
        __syncthreads();
        {
            double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k0 = 0; k0 < KZ; k0 += PG) {
                if (k0 < nk) {
                    T a[PG], D[PG];
                    product(k0, [&](int k) -> T { return r[k]; }, zr[0], zr[1], a, D, t);
#pragma unroll
                    for (int e = 0; e < PG; ++e) {
                        const double ae = (double)a[e], s = (double)D[e] * (double)r[k0 + e];
                        const double sh = (double)rt[k0 + e];
                        acc[0] += ae * s;
                        acc[1] += ae * ae;
                        acc[2] += s * s;
                        acc[3] += sh * s;
                        acc[4] += sh * ae;
                    }
                }
                if constexpr (KZ > 8) __builtin_amdgcn_sched_barrier(0);
            }
            publish(ph, t, acc);
        }
        ++ph;
        // previous-iteration slots of fin_b
        sc.alpha[1] = alpha;
        sc.rho[1] = rho;
        sc.iter[1] = iter;
        fresh = false;
    }

    // the iterate and the outcome
    if constexpr (BIG) {
        if (upx) update_x();
#pragma unroll
        for (int k = 0; k < KZ; ++k) {
            T x;
            xfetch(xx, xat, k * XP, x);
            if (act && k < nk) gX[g0 + (unsigned)P * k] = x;
        }
    } else {
#pragma unroll
        for (int k = 0; k < KZ; ++k)
            if (act && k < nk) gX[g0 + (unsigned)P * k] = xr[BIG ? 0 : k];
    }
    if (lb == 0 && tid == 0) {
        Scalars *o = S.sc;
        o->rr = rr;
        o->iter[0] = o->iter[1] = iter;
        o->iter_done = iter;
        o->fresh = 0;
        o->stop_a = stop;
        o->stop = stop;
    }
}

// The scalar block of a start.
template <typename T>
__device__ __forceinline__ void start_sys(const ChipSys<T> &S)
{
    constexpr unsigned WS = sizeof(Scalars) / 4;
    if (threadIdx.x < WS)
        reinterpret_cast<unsigned *>(S.sc)[threadIdx.x] = reinterpret_cast<const unsigned *>(&S.init)[threadIdx.x];
}

template <typename T>
__global__ __launch_bounds__(256) void k_chip_start1(ChipSys<T> one, ChipSys<T> *table)
{
    start_sys(one);
    constexpr unsigned W = sizeof(ChipSys<T>) / 4;
    static_assert(sizeof(ChipSys<T>) % 4 == 0 && W <= 256, "one word per thread of the first workgroup");
    if (threadIdx.x < W)
        reinterpret_cast<unsigned *>(table)[threadIdx.x] = reinterpret_cast<const unsigned *>(&one)[threadIdx.x];
}

template <typename T>
__global__ __launch_bounds__(256) void k_chip_start(const ChipSys<T> *table)
{
    start_sys(table[blockIdx.x]);
}

// ------------------------------------------------------------------ host

size_t chip_lds(int kz, size_t elem)
{
    return ((size_t)kz * CH_LP + FTAB + PAL_MAX + (kz > 8 ? (size_t)kz * CH_NT : 0)) * elem;
}

ChipSpace chip_space(const ChipGeom &ge, int kz, size_t elem)
{
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t values = (size_t)2 * ge.G * ge.fstride;   // two buffers of boundary values
    ChipSpace m{};
    if (kz <= 8) {
        m.face = al(CH_SUMS);
        m.tagged = m.face + al(values * 2 * elem);
    } else {
        m.tagged = al(CH_SUMS);
        m.xtile = al(values * elem);
        m.plain = m.xtile + (size_t)ge.G * kz * CH_NT * elem;
    }
    return m;
}

// Among the partitions that fit, the one of least cost: a tile's time for its
// planes (one wave per SIMD works on 256 columns at a time: about 500 cycles
// a plane and iteration, twice that with 16 planes a tile) and the exchange of the sums among the tiles (about
// 21 cycles per tile and iteration, 33^3 with 64 and 256 tiles), then the
// fewest xy halo nodes.
ChipGeom chip_partition(int nx, int ny, int nz, int neu, int gcap, int kzmax)
{
    ChipGeom best;
    const int n[3] = {nx, ny, nz};
    int o[3], u[3];
    for (int a = 0; a < 3; ++a) {
        o[a] = ((neu >> (2 * a)) & 1) ? 0 : 1;
        u[a] = n[a] - o[a] - (((neu >> (2 * a + 1)) & 1) ? 0 : 1);
        if (u[a] < 1) return best;
    }
    gcap = gcap < CH_GMAX ? gcap : CH_GMAX;
    // a face takes whole 128-byte lines: a line has one writer and one reader
    auto pad = [](int e) { return (e + 31) / 32 * 32; };
    long bcost = -1;
    for (int cz = (u[2] + kzmax - 1) / kzmax; cz <= u[2] && cz <= gcap; ++cz) {
        const int bz = (u[2] + cz - 1) / cz;
        const int kz = bz <= 4 ? 4 : bz <= 8 ? 8 : 16;
        for (int cy = 1; cy <= u[1] && cy * cz <= gcap; ++cy) {
            const int by = (u[1] + cy - 1) / cy;
            if (by > CH_NT || (cy > 1 && u[1] / cy < 2)) continue;
            for (int cx = 1; cx <= u[0] && cx * cy * cz <= gcap; ++cx) {
                const int bx = (u[0] + cx - 1) / cx;
                if (bx * by > CH_NT || (cx > 1 && u[0] / cx < 2)) continue;
                if ((bx + 2) * (by + 2) > CH_LP - 1 || 2 * (bx + by) * bz > chip_halo_slots(kz) * CH_NT) continue;
                if (2 * (pad(by * bz) + pad(bx * bz) + pad(bx * by)) > chip_face_slots(kz) * CH_NT) continue;
                const long rows = (bx * by + 255) / 256, planes = bz <= 4 ? (bz + 1) / 2 * 2 : (bz + 3) / 4 * (kz > 8 ? 8 : 4);
                const long cost = (rows * planes * 24 + cx * cy * cz) * 4096 + 2 * (bx + by) * bz;
                if (bcost >= 0 && cost >= bcost) continue;
                bcost = cost;
                best.KZ = kz;
                for (int a = 0; a < 3; ++a) { best.o[a] = o[a]; best.n[a] = u[a]; }
                best.c[0] = cx; best.c[1] = cy; best.c[2] = cz;
                best.G = cx * cy * cz;
                best.fx = pad(by * bz); best.fy = pad(bx * bz); best.fz = pad(bx * by);
                best.fstride = 2 * (best.fx + best.fy + best.fz);
            }
        }
    }
    return best;
}

template <typename T>
hipError_t chip_start(const ChipSys<T> *one, ChipSys<T> *table, int nsys, hipStream_t s)
{
    if (one) hipLaunchKernelGGL((k_chip_start1<T>), dim3(1), dim3(256), 0, s, *one, table);
    else hipLaunchKernelGGL((k_chip_start<T>), dim3(nsys), dim3(256), 0, s, (const ChipSys<T> *)table);
    return hipGetLastError();
}

template <typename T, int FORM, int KZ>
static hipError_t launch_k(const ChipSys<T> *table, const int *first, int nsys, int tiles, hipStream_t s)
{
    auto kern = k_chip<T, FORM, KZ>;
    const size_t lds = chip_lds(KZ, sizeof(T));
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(CH_NT), lds, s, table, first, nsys);
    return hipGetLastError();
}

template <typename T>
hipError_t chip_launch(int form, int kz, const ChipSys<T> *table, const int *first, int nsys, int tiles, hipStream_t s)
{
    switch (form * 100 + kz) {
    case CHF_CEPS * 100 + 4: return launch_k<T, CHF_CEPS, 4>(table, first, nsys, tiles, s);
    case CHF_CEPS * 100 + 8: return launch_k<T, CHF_CEPS, 8>(table, first, nsys, tiles, s);
    case CHF_CEPS * 100 + 16: return launch_k<T, CHF_CEPS, 16>(table, first, nsys, tiles, s);
    case CHF_NONE * 100 + 4: return launch_k<T, CHF_NONE, 4>(table, first, nsys, tiles, s);
    case CHF_NONE * 100 + 8: return launch_k<T, CHF_NONE, 8>(table, first, nsys, tiles, s);
    case CHF_NONE * 100 + 16: return launch_k<T, CHF_NONE, 16>(table, first, nsys, tiles, s);
    case CHF_NODE * 100 + 4: return launch_k<T, CHF_NODE, 4>(table, first, nsys, tiles, s);
    case CHF_NODE * 100 + 8: return launch_k<T, CHF_NODE, 8>(table, first, nsys, tiles, s);
    case CHF_CLASS * 100 + 4: return launch_k<T, CHF_CLASS, 4>(table, first, nsys, tiles, s);
    case CHF_CLASS * 100 + 8: return launch_k<T, CHF_CLASS, 8>(table, first, nsys, tiles, s);
    case CHF_CLASS * 100 + 16: return launch_k<T, CHF_CLASS, 16>(table, first, nsys, tiles, s);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t chip_start<double>(const ChipSys<double> *, ChipSys<double> *, int, hipStream_t);
template hipError_t chip_start<float>(const ChipSys<float> *, ChipSys<float> *, int, hipStream_t);
template hipError_t chip_launch<double>(int, int, const ChipSys<double> *, const int *, int, int, hipStream_t);
template hipError_t chip_launch<float>(int, int, const ChipSys<float> *, const int *, int, int, hipStream_t);

}  // namespace pfk
