// Image pre-processing before a two-fluid simulation of a segmented rock image (section
// "Initial conditions and wetting maps"; the mixing region of section "Simulation protocol for
// steady-state flow"): an exact squared Euclidean distance transform, the morphological
// drainage built on it (sphere-placing, Adalsteinsson and Hilpert 2006), the mixed-wet
// relabelling of solid voxels near the drained fluid, and the mixing layer that opens the
// inlet and outlet planes to each other.
//
// Distance transform, separable: the squared distance to the nearest feature voxel is
// min over (y', z') of [g(x; y', z')^2 + (y - y')^2 + (z - z')^2], g the distance along the
// row. The row pass finds g from the rows packed as 64-voxel bit words (windows of 32 voxels to each
// side, then find-first-set on whole words); the y and z passes search outward from each voxel and
// stop once d^2 reaches the best value so far, which is exact because every candidate at offset d
// costs at least d^2. A thread of those passes takes 8 positions of a line and reads the 24 values of
// their offsets up to 8 at once, so the common short search is one round trip. With a cap c (only
// distances below c matter) every value is clipped at c and the searches stop at c. Squared
// distances are int32 with kInf = 2^30 - 1 for "none": sizes up to 16384 keep kInf + n^2 below 2^31.
//
// Per-voxel kernels run on a 2-D grid: blockIdx.x is the image row (y, z), blockIdx.y the
// chunk of x, so no thread divides a 64-bit index. Bit rows are packed with wide loads and
// shuffles when rows are a multiple of 8 long, else with a ballot per word.
//
// Connectivity of the sphere centres to the inlet plane: union-find labelling of the runs of
// centres along x, a run's label at its first voxel; runs that touch across a -y or
// -z face (or the periodic x face) are united by linking the larger root under the smaller
// with atomicMin, retrying from the new parent when another thread linked first. A parent
// index is never larger than its child, so every find walks a strictly decreasing chain and
// ends. After the merges the roots of the runs in the z = 0 plane are flagged, and a centre is
// reached when its run's root is flagged. Counts use fixed-shape workgroup
// sums and a fixed-order final sum, so every result is deterministic.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "lbm_domain.h"

using namespace lbm;

namespace {

constexpr int32_t kInf = 0x3fffffff;
constexpr int kMaxDim = 16384;
constexpr int kPrepThreads = 256;
constexpr int kSumThreads = 1024;

struct Box {
    int nx, ny, nz, W;   // W: 64-bit words per row
    int64_t nvox;        // nx*ny*nz
    int64_t nwords;      // ny*nz*W
    int per;             // bit a: axis a periodic
    int tpb;             // threads per workgroup of the per-voxel kernels
    int chunks;          // workgroups per row
};

// ---------------------------------------------------------------------------------------------
// Kernels

// The voxel of this thread in the 2-D grid of the per-voxel kernels.
struct VoxelIdx {
    int64_t v;
    int row, x;
    bool active;
};

__device__ __forceinline__ VoxelIdx voxel_of(const Box& b) {
    VoxelIdx r;
    r.row = (int)blockIdx.x;
    r.x = (int)blockIdx.y * (int)blockDim.x + (int)threadIdx.x;
    r.active = r.x < b.nx;
    r.v = (int64_t)r.row * b.nx + r.x;
    return r;
}

struct FeatureNonzero {
    const uint8_t* m;
    __device__ bool operator()(int64_t v) const { return m[v] != 0; }
};
struct FeatureZero {
    const uint8_t* m;
    __device__ bool operator()(int64_t v) const { return m[v] == 0; }
};
struct FeatureCentre {   // pore voxel where a sphere of squared radius k fits
    const uint8_t* pore;
    const int32_t* d2;
    int32_t k;
    __device__ bool operator()(int64_t v) const { return pore[v] != 0 && d2[v] >= k; }
};
// Four consecutive 64-voxel words per wave (their loads in flight together): lane i holds bit i
// of each (x = 64 w + i of the word's row).
constexpr int kWordsPerWave = 4;

template <typename P>
__global__ void __launch_bounds__(256) pack_kernel(Box b, P pred, uint64_t* __restrict__ bits) {
    const int64_t word0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kWordsPerWave;
    const int lane = threadIdx.x & 63;
    if (word0 >= b.nwords) return;   // the whole wave
    bool p[kWordsPerWave];
#pragma unroll
    for (int j = 0; j < kWordsPerWave; ++j) {
        const int64_t word = word0 + j;
        const int row = (int)(word / b.W);
        const int x = 64 * (int)(word - (int64_t)row * b.W) + lane;
        p[j] = word < b.nwords && x < b.nx && pred((int64_t)row * b.nx + x);
    }
#pragma unroll
    for (int j = 0; j < kWordsPerWave; ++j) {
        const uint64_t m = __ballot(p[j]);
        if (lane == j && word0 + j < b.nwords) bits[word0 + j] = m;
    }
}

// Rows whose length is a multiple of 8: each lane reads 8 consecutive voxels with wide loads
// (8-byte and 16-byte aligned) and the 8 lanes of a word merge their bytes by shuffles; a wave
// covers 8 words. The predicate's byte8(v) gives bit i for voxel v + i.
__device__ __forceinline__ uint32_t nonzero_bytes(uint64_t w) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) m |= (((w >> (8 * i)) & 0xffull) != 0 ? 1u : 0u) << i;
    return m;
}
struct Wide8Nonzero {
    const uint8_t* m;
    __device__ uint32_t byte8(int64_t v) const {
        return nonzero_bytes(*reinterpret_cast<const uint64_t*>(m + v));
    }
};
struct Wide8Zero {
    const uint8_t* m;
    __device__ uint32_t byte8(int64_t v) const {
        return ~nonzero_bytes(*reinterpret_cast<const uint64_t*>(m + v)) & 0xffu;
    }
};
struct Wide8Centre {
    const uint8_t* pore;
    const int32_t* d2;
    int32_t k;
    __device__ uint32_t byte8(int64_t v) const {
        const uint32_t pm = nonzero_bytes(*reinterpret_cast<const uint64_t*>(pore + v));
        const int4 a = *reinterpret_cast<const int4*>(d2 + v);
        const int4 c = *reinterpret_cast<const int4*>(d2 + v + 4);
        const uint32_t dm = (a.x >= k ? 1u : 0u) | (a.y >= k ? 2u : 0u) | (a.z >= k ? 4u : 0u) |
                            (a.w >= k ? 8u : 0u) | (c.x >= k ? 16u : 0u) | (c.y >= k ? 32u : 0u) |
                            (c.z >= k ? 64u : 0u) | (c.w >= k ? 128u : 0u);
        return pm & dm;
    }
};

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int mask) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, mask);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), mask);
    return ((uint64_t)hi << 32) | lo;
}

template <typename P>
__global__ void __launch_bounds__(256) pack8_kernel(Box b, P pred, uint64_t* __restrict__ bits) {
    const int lane = threadIdx.x & 63;
    const int g = lane & 7;
    const int64_t word = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 8 + (lane >> 3);
    uint32_t byte = 0;
    if (word < b.nwords) {
        const int row = (int)(word / b.W);
        const int x = 64 * (int)(word - (int64_t)row * b.W) + 8 * g;
        if (x < b.nx) byte = pred.byte8((int64_t)row * b.nx + x);
    }
    uint64_t m = (uint64_t)byte << (8 * g);
    m |= shfl_xor_u64(m, 1);
    m |= shfl_xor_u64(m, 2);
    m |= shfl_xor_u64(m, 4);
    if (g == 0 && word < b.nwords) bits[word] = m;
}

// Complement of row bits within each row (bits past nx stay clear).
__global__ void __launch_bounds__(256) invert_bits_kernel(Box b, const uint64_t* __restrict__ in,
                                                          uint64_t* __restrict__ out) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= b.nwords) return;
    const int w = (int)(k % b.W);
    const int tail = b.nx & 63;
    const uint64_t valid = (w == b.W - 1 && tail) ? ((1ull << tail) - 1ull) : ~0ull;
    out[k] = ~in[k] & valid;
}

// First set bit at a position in [p, e] of a row (p <= e), or -1.
__device__ __forceinline__ int first_set(const uint64_t* __restrict__ r, int p, int e) {
    int w = p >> 6;
    const int we = e >> 6;
    uint64_t m = r[w] & (~0ull << (p & 63));
    while (true) {
        if (w == we) {
            const int eb = e & 63;
            if (eb != 63) m &= (1ull << (eb + 1)) - 1ull;
            return m ? (w << 6) + __ffsll((long long)m) - 1 : -1;
        }
        if (m) return (w << 6) + __ffsll((long long)m) - 1;
        m = r[++w];
    }
}

// Last set bit at a position in [s, p] of a row (s <= p), or -1.
__device__ __forceinline__ int last_set(const uint64_t* __restrict__ r, int s, int p) {
    int w = p >> 6;
    const int ws = s >> 6;
    const int pb = p & 63;
    uint64_t m = r[w] & (pb == 63 ? ~0ull : ((1ull << (pb + 1)) - 1ull));
    while (true) {
        if (w == ws) {
            m &= ~0ull << (s & 63);
            return m ? (w << 6) + 63 - __clzll((long long)m) : -1;
        }
        if (m) return (w << 6) + 63 - __clzll((long long)m);
        m = r[--w];
    }
}

// Row pass: out[v] = min(g^2, cap), g = distance along x to the nearest feature bit in the
// row (wrapping when x is periodic), searched to at most `lim` voxels. Four consecutive voxels
// per thread (one 16-byte store when nx is a multiple of 4). row_dist: the distance from the
// words w-1, w, w+1 around a voxel where they settle it; the full word-by-word search runs only
// for a side they leave open and whose remainder lies within the limit.
__device__ __forceinline__ int row_dist(const uint64_t* __restrict__ r, int W, int nx, bool per,
                                        int lim, int x, uint64_t cur, uint64_t lo, uint64_t hi) {
    const int w = x >> 6, sh = x & 63;
    int d = kInf;
    bool right_open = false, left_open = false;
    // right: bits >= x in this word, then the next word
    const uint64_t rc = cur >> sh;
    if (rc) {
        d = __ffsll((long long)rc) - 1;
    } else if (hi) {
        d = 64 - sh + __ffsll((long long)hi) - 1;
    } else {
        right_open = true;
    }
    // left: bits <= x in this word, then the previous word
    const uint64_t lc = sh == 63 ? cur : (cur & ((1ull << (sh + 1)) - 1ull));
    if (lc) {
        d = min(d, sh - (63 - __clzll((long long)lc)));
    } else if (lo) {
        d = min(d, sh + 1 + __clzll((long long)lo));
    } else {
        left_open = true;
    }
    // A hit is the nearest feature on its side without wrapping, so it is never worse than a
    // wrapped one on that side; a hit beyond lim gives d^2 > cap (capped) or is matched by the
    // search on the other side (periodic), so the result is min(d^2, cap) either way. An open
    // side is searched in full only when what lies beyond the window (a further word, or the
    // wrap through the periodic face) is within the limit and could still be nearer than d.
    int rb = w + 1 < W ? 128 - sh : kInf;
    int lb = w > 0 ? sh + 65 : kInf;
    if (per) {
        rb = min(rb, nx - x);
        lb = min(lb, x + 1);
    }
    if (right_open && rb <= lim && d > rb) {
        int q = first_set(r, x, min(nx - 1, x + lim));
        if (q >= 0) {
            d = min(d, q - x);
        } else if (per && x + lim >= nx && x > 0) {
            q = first_set(r, 0, min(x - 1, x + lim - nx));
            if (q >= 0) d = min(d, q + nx - x);
        }
    }
    if (left_open && lb <= lim && d > lb) {
        int q = last_set(r, max(0, x - lim), x);
        if (q >= 0) {
            d = min(d, x - q);
        } else if (per && x - lim < 0 && x < nx - 1) {
            q = last_set(r, max(x + 1, x - lim + nx), nx - 1);
            if (q >= 0) d = min(d, x + nx - q);
        }
    }
    return d;
}

// Squared distances along x, at most cap, of the four voxels from x0 (a multiple of 4) of the row
// whose words are r.
__device__ __forceinline__ void row_quad(const Box& b, const uint64_t* __restrict__ r, int x0,
                                         int lim, int32_t cap, int (&res)[4]) {
    const bool per = (b.per & 1) != 0;
    // The half words at and beside the four voxels (which share one) settle every distance below
    // 32, in about fifteen instructions without a branch; row_dist with its three words and
    // searches takes over five times as many, and was what bound this pass (256^3, bytes: 56 us;
    // now 22). On a periodic row the windows near the ends go on with the first and the last
    // 32 voxels of the row, which settles every distance on a row shorter than 64 (left to row_dist,
    // such rows took the byte pass of 48^3 from 6.9 to 8.5 us).
    const uint32_t* h = reinterpret_cast<const uint32_t*>(r);
    const int k = x0 >> 5;
    const uint64_t cur = h[k], lo = k > 0 ? h[k - 1] : 0u, hi = k + 1 < 2 * b.W ? h[k + 1] : 0u;
    const uint64_t right = hi << 32 | cur, left = cur << 32 | lo;
    uint32_t head = 0, last = 0;
    if (per) {
        const int e = (b.nx - 1) >> 5;
        head = h[0];
        last = (uint32_t)(((uint64_t)h[e] << 32 | (e > 0 ? h[e - 1] : 0u)) >>
                          (((b.nx - 1) & 31) + 1));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int x = x0 + j, sh = x & 31;
        uint32_t R = (uint32_t)(right >> sh), L = (uint32_t)(left >> (sh + 1));
        if (per) {
            if (b.nx - x < 32) R |= head << max(0, b.nx - x);
            if (x < 31) L |= last >> (x + 1);
        }
        int d = min(R ? __ffs((int)R) - 1 : 32, L ? __clz((int)L) : 32);
        const bool more = d == 32 && lim >= 32;
        if (d == 32) d = kInf;
        if (more && x < b.nx) {
            const int w = x0 >> 6;
            d = row_dist(r, b.W, b.nx, per, lim, x, r[w], w > 0 ? r[w - 1] : 0ull,
                         w + 1 < b.W ? r[w + 1] : 0ull);
        }
        res[j] = d >= kInf ? cap : min(d * d, cap);
    }
}

// A workgroup takes 256 >> qshift rows, with 1 << qshift threads (at least the row's quads, at
// most 256) for each: one row to a workgroup left most of its threads idle and was bound by the
// rate at which workgroups start (128^3: 16384 of one wave, 10.3 us; now 2048, 5.9 us).
template <typename T>
__global__ void __launch_bounds__(256) edt_row_kernel(Box b, const uint64_t* __restrict__ bits,
                                                      int qshift, int lim, int32_t cap,
                                                      T* __restrict__ out) {
    const int row = (int)blockIdx.x * (256 >> qshift) + ((int)threadIdx.x >> qshift);
    const int x0 = 4 * (((int)blockIdx.y << qshift) + ((int)threadIdx.x & ((1 << qshift) - 1)));
    if (x0 >= b.nx || row >= b.ny * b.nz) return;
    int res[4];
    row_quad(b, bits + (int64_t)row * b.W, x0, lim, cap, res);
    const int64_t v = (int64_t)row * b.nx + x0;
    if ((b.nx & 3) == 0) {
        if constexpr (sizeof(T) == 4)
            *reinterpret_cast<int4*>(out + v) = make_int4(res[0], res[1], res[2], res[3]);
        else
            *reinterpret_cast<uchar4*>(out + v) =
                make_uchar4((unsigned char)res[0], (unsigned char)res[1], (unsigned char)res[2],
                            (unsigned char)res[3]);
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (x0 + j < b.nx) out[v + j] = (T)res[j];
    }
}

// Continues min over d >= d0 of in[base + ((c + d) mod n) stride] + d^2 from `best`, stopping once
// d^2 reaches best. Four offsets to a round trip: an offset more than needed, and the place c
// itself in the stead of one outside the line, give terms that are never below the minimum.
template <typename T>
__device__ __forceinline__ int line_min_from(const T* __restrict__ in, int64_t base,
                                             int64_t stride, int c, int n, bool per, int best,
                                             int d0) {
    const int lim = per ? n / 2 : max(c, n - 1 - c);
    for (int d = d0; d <= lim; d += 4) {
        if (d * d >= best) break;
        int v[8];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            int a = c + d + k, e = c - d - k;
            if (per) {
                a = a >= n ? a - n : a;
                e = e < 0 ? e + n : e;
            }
            if (a >= n) a = c;
            if (e < 0) e = c;
            v[2 * k] = (int)in[base + (int64_t)a * stride];
            v[2 * k + 1] = (int)in[base + (int64_t)e * stride];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            best = min(best, min(v[2 * k], v[2 * k + 1]) + (d + k) * (d + k));
    }
    return best;
}

__device__ __forceinline__ int wall_min(const Box& b, int walls, int x, int y, int z, int best) {
    const int cx[3] = {x, y, z};
    const int nn[3] = {b.nx, b.ny, b.nz};
#pragma unroll
    for (int a = 0; a < 3; ++a)
        if (((walls >> a) & 1) && !((b.per >> a) & 1)) {
            const int lo = cx[a] + 1, hi = nn[a] - cx[a];
            best = min(best, min(lo * lo, hi * hi));
        }
    return best;
}

// Line pass along axis `ax` (1: y, 2: z) over kSeg consecutive positions c0 .. c0+kSeg-1 of one
// line per thread: the window in[c0-kWin .. c0+kSeg+kWin-1] is read at once (an unconditional
// load for each place, the ones outside a non-periodic line replaced afterwards), so offsets up
// to kWin cost no further load, and larger ones (only where the best value so far exceeds
// (kWin + 1)^2) continue from memory, one dependent round trip per offset. kWin was 4 with a
// branch around each load: the continuation then ran in most waves of a rock image, whose pore
// bodies are 5 to 8 voxels wide (128^3: 10.3 us a pass; now 7.4; the z pass with the wall terms 10.6). A window value of a wrapped
// position further than half a period is an upper bound of that position's term, never below the
// minimum, so it may stay in.
//   MODE 0: out[v] = min(cap, best), with the wall-plane terms of `walls`;
//   MODE 2: the same without a cap, -1 where there is no feature (the last pass of a transform
//           that is the result);
//   MODE 1 (z pass of the drainage dilation): a pore voxel is non-wetting when best < cap (the
//           squared radius); writes nw when it is not null and the count of each workgroup
//           (kPrepThreads threads).
constexpr int kSeg = 8;
constexpr int kWin = 8;

// The places of a window's entries, each given to `load` with its index. A periodic line is walked
// from where the window begins: one remainder for the window, where one for each entry beyond the
// ends took a fifth of a short line's pass. Any place (c0) stands for one outside another line.
template <typename Load>
__device__ __forceinline__ void window_places(int c0, int n, bool per, Load load) {
    if (per) {
        int c = c0 < kWin ? (n - (kWin - c0) % n) % n : c0 - kWin;
#pragma unroll
        for (int j = 0; j < kSeg + 2 * kWin; ++j) {
            load(j, c);
            c = c + 1 < n ? c + 1 : 0;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kSeg + 2 * kWin; ++j) {
            const int c = c0 - kWin + j;
            load(j, c < 0 || c >= n ? c0 : c);
        }
    }
}

// The least of a window's values seen from its place i, with best.
__device__ __forceinline__ int window_min(const int (&win)[kSeg + 2 * kWin], int i, int best) {
#pragma unroll
    for (int d = 1; d <= kWin; ++d)
        best = min(best, min(win[i + kWin + d], win[i + kWin - d]) + d * d);
    return best;
}

template <int MODE, typename T>
__global__ void __launch_bounds__(256) edt_seg_kernel(Box b, int ax, int32_t cap, int walls,
                                                      const T* __restrict__ in,
                                                      T* __restrict__ out,
                                                      const uint8_t* __restrict__ pore,
                                                      uint8_t* __restrict__ nw,
                                                      int* __restrict__ part) {
    const int x = (int)blockIdx.y * (int)blockDim.x + (int)threadIdx.x;
    const bool active = x < b.nx;
    const int n = ax == 1 ? b.ny : b.nz;
    const int nseg = (n + kSeg - 1) / kSeg;
    const int seg = (int)blockIdx.x % nseg;
    const int o = (int)blockIdx.x / nseg;   // z when ax == 1, y when ax == 2
    const int64_t stride = ax == 1 ? (int64_t)b.nx : (int64_t)b.nx * b.ny;
    const int64_t base = ax == 1 ? (int64_t)o * b.ny * b.nx + x : (int64_t)o * b.nx + x;
    const bool per = ((b.per >> ax) & 1) != 0;
    const int c0 = seg * kSeg;
    int cnt = 0;
    if (active) {
        int win[kSeg + 2 * kWin];
        window_places(c0, n, per, [&](int j, int c) {
            win[j] = (int)in[base + (int64_t)c * stride];
        });
        if (!per) {
#pragma unroll
            for (int j = 0; j < kSeg + 2 * kWin; ++j)
                if (c0 - kWin + j < 0 || c0 - kWin + j >= n) win[j] = kInf;
        }
#pragma unroll
        for (int i = 0; i < kSeg; ++i) {
            const int c = c0 + i;
            if (c >= n) break;
            const int64_t v = base + (int64_t)c * stride;
            if (MODE == 1 && !pore[v]) {
                if (nw) nw[v] = 0;
                continue;
            }
            int best = win[i + kWin];
            if (walls) best = wall_min(b, walls, x, ax == 1 ? c : o, ax == 1 ? o : c, best);
            best = window_min(win, i, best);
            if (best > (kWin + 1) * (kWin + 1))
                best = line_min_from(in, base, stride, c, n, per, best, kWin + 1);
            if (MODE == 0) {
                out[v] = (T)min(best, cap);
            } else if (MODE == 2) {
                out[v] = best >= kInf ? (T)-1 : (T)best;
            } else {
                const bool f = best < cap;
                cnt += f ? 1 : 0;
                if (nw) nw[v] = f ? 1 : 0;
            }
        }
    }
    if (MODE == 1) {
        for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
        __shared__ int ws[kPrepThreads / 64];
        if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = cnt;
        __syncthreads();
        if (threadIdx.x == 0) {
            int t = 0;
            for (int i = 0; i < kPrepThreads / 64; ++i) t += ws[i];
            part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
        }
    }
}

// The row and y passes of int32 distances in one: a workgroup takes 64 columns of a plane, whose
// row distances stay in LDS for the y pass, so they are neither written nor read again, and the
// second pass has no launch. kWin rows before and after the plane's hold what lies beyond its
// faces, so that the windows need no tests. Bound by the latency of its few workgroups at 128^3 (one
// of 16 waves a CU), by instructions from 256^3. Row pass and y pass against this, 10% features:
// 128^3 5.9 + 10 us and a launch, now 10 (a whole transform 26.5 -> 21.8); 256^3 25 + 44, now 44;
// 352^3 67 + 112, now 127; 480^3 141 + 253, now 287.
constexpr int kPlaneThreads = 1024, kPlaneCols = 64, kPlaneLd = 68, kPlaneRows = 480;
// Whether the passes are taken in one (the tile fits the LDS to 480 rows):
//  * up to one workgroup a CU, planes of at most 128 rows: the launch that is saved counts (whole
//    transforms: 64^3 15.0 -> 11.5 us, 256 planes of 64 x 8 13.9 -> 11.0, of 60 x 64 23.2 -> 17.1),
//    while a single plane of 480 rows would take 20 us against 6;
//  * more of them, planes of at least 96 rows, which give each of the 16 waves its rows: 240 planes'
//    columns of 256 rows 16 us against 20, 1000 of 96 rows 47.2 against 48.4. With fewer rows most
//    waves idle (1000 planes of 124 x 32 50 us against 42.5, 8192 of 60 x 8 89 against 44).
bool plane_pass(const Box& b) {
    const int64_t groups = (int64_t)b.nz * ((b.nx + kPlaneCols - 1) / kPlaneCols);
    return groups <= 256 ? b.ny <= 128 || (b.ny <= kPlaneRows && groups >= 240)
                         : b.ny >= 96 && b.ny <= kPlaneRows;
}
// BYTES: the features are given as the image's bytes (rows of a multiple of 8, 8-byte aligned) and
// the workgroup packs its plane's words into LDS itself, which saves a launch (a whole transform of
// 64^3 11.5 -> 9.5 us, of 128^3 21.8 -> 20.5, of 60 planes of 256 x 256 34.2 -> 32.2). Every workgroup
// of a plane does so: rows of up to kPlaneBytes, four workgroups.
constexpr int kPlaneBytes = 256;
__host__ __device__ inline int plane_rows(const Box& b) {   // of the tile
    return (b.ny + kSeg - 1) / kSeg * kSeg + 2 * kWin;
}
template <bool BYTES>
__global__ void __launch_bounds__(kPlaneThreads) edt_plane_kernel(Box b,
                                                                  const uint64_t* __restrict__ bits,
                                                                  const uint8_t* __restrict__ image,
                                                                  int lim, int32_t cap,
                                                                  int32_t* __restrict__ out) {
    extern __shared__ int4 plane[];
    int32_t* val = reinterpret_cast<int32_t*>(plane) + kWin * kPlaneLd;   // row y = 0
    uint64_t* words = reinterpret_cast<uint64_t*>(val + (plane_rows(b) - kWin) * kPlaneLd);
    const int t = (int)threadIdx.x, chunks = (b.nx + kPlaneCols - 1) / kPlaneCols;
    const int z = (int)blockIdx.x / chunks, xc = ((int)blockIdx.x - z * chunks) * kPlaneCols;
    const int q = 4 * (t & 15), rows = plane_rows(b) - 2 * kWin;
    const bool per = (b.per & 2) != 0;
    if (BYTES) {
        const uint8_t* in = image + (int64_t)z * b.ny * b.nx;
        for (int i = t; i < 8 * b.W * b.ny; i += kPlaneThreads) {
            const int y = i / (8 * b.W), x = 8 * (i - y * 8 * b.W);
            reinterpret_cast<uint8_t*>(words)[i] =
                x < b.nx ? (uint8_t)Wide8Nonzero{in}.byte8((int64_t)y * b.nx + x) : 0;
        }
        __syncthreads();
    }
    if (xc + q < b.nx) {
        for (int y = (t >> 4) - kWin; y < rows + kWin; y += kPlaneThreads / 16) {
            const bool beyond = y < 0 || y >= b.ny;
            int res[4] = {kInf, kInf, kInf, kInf};
            int x0 = xc + q;
            asm volatile("" : "+v"(x0));   // or what depends on x alone is held over all rows
            if (!beyond || per) {
                const int c = beyond ? ((y % b.ny) + b.ny) % b.ny : y;
                if (BYTES)
                    row_quad(b, words + c * b.W, x0, lim, cap, res);
                else
                    row_quad(b, bits + ((int64_t)z * b.ny + c) * b.W, x0, lim, cap, res);
            }
            *reinterpret_cast<int4*>(val + y * kPlaneLd + q) =
                make_int4(res[0], res[1], res[2], res[3]);
        }
    }
    __syncthreads();
    const int col = t & 63, x = xc + col;
    if (x >= b.nx) return;
    for (int c0 = kSeg * __builtin_amdgcn_readfirstlane(t >> 6); c0 < b.ny;
         c0 += kSeg * (kPlaneThreads / 64)) {
        int win[kSeg + 2 * kWin];
#pragma unroll
        for (int j = 0; j < kSeg + 2 * kWin; ++j) win[j] = val[(c0 - kWin + j) * kPlaneLd + col];
#pragma unroll
        for (int i = 0; i < kSeg; ++i) {
            const int c = c0 + i;
            if (c >= b.ny) break;
            int best = window_min(win, i, win[i + kWin]);
            if (best > (kWin + 1) * (kWin + 1))
                best = line_min_from(val, col, kPlaneLd, c, b.ny, per, best, kWin + 1);
            out[((int64_t)z * b.ny + c) * b.nx + x] = min(best, cap);
        }
    }
}

// The line pass for distances held in bytes (cap <= 255), rows of a multiple of 4 and images of
// kQuadVoxels and more: a thread
// takes four neighbouring lines, a window entry is one 4-byte load, and the minima run on pairs
// of 16-bit values. With a byte per load and a minimum per value the passes took as long as with
// int32 (256^3: 43 us each, bound by their loads and instructions); now 23. The lines'
// threads are 1 << qshift to a row as in the row pass, so a workgroup holds 256 >> qshift
// segments. MODE 0 and 1 as above. Offsets beyond the window matter only to a cap above
// (kWin + 1)^2.
typedef unsigned short Pair16 __attribute__((ext_vector_type(2)));

template <int MODE>
__global__ void __launch_bounds__(256) edt_seg8_kernel(Box b, int ax, int qshift, int32_t cap,
                                                       int walls, const uint8_t* __restrict__ in,
                                                       uint8_t* __restrict__ out,
                                                       const uint8_t* __restrict__ pore,
                                                       uint8_t* __restrict__ nw,
                                                       int* __restrict__ part) {
    constexpr unsigned short kFar = 0x7fff;   // no value: above every cap, also with d^2 added
    const int x0 = 4 * (((int)blockIdx.y << qshift) + ((int)threadIdx.x & ((1 << qshift) - 1)));
    const int n = ax == 1 ? b.ny : b.nz, other = ax == 1 ? b.nz : b.ny;
    const int nseg = (n + kSeg - 1) / kSeg;
    const int at = (int)blockIdx.x * (256 >> qshift) + ((int)threadIdx.x >> qshift);
    const int o = at / nseg, c0 = (at - o * nseg) * kSeg;
    const int64_t stride = ax == 1 ? (int64_t)b.nx : (int64_t)b.nx * b.ny;
    const int64_t base = ax == 1 ? (int64_t)o * b.ny * b.nx + x0 : (int64_t)o * b.nx + x0;
    const bool per = ((b.per >> ax) & 1) != 0;
    int cnt = 0;
    if (x0 < b.nx && at < other * nseg) {
        uint32_t raw[kSeg + 2 * kWin];
        window_places(c0, n, per, [&](int j, int c) {
            raw[j] = *reinterpret_cast<const uint32_t*>(in + base + (int64_t)c * stride);
        });
        Pair16 even[kSeg + 2 * kWin], odd[kSeg + 2 * kWin];   // lines x0, x0 + 2 and x0 + 1, x0 + 3
#pragma unroll
        for (int j = 0; j < kSeg + 2 * kWin; ++j) {
            const int c = c0 - kWin + j;
            const bool none = !per && (c < 0 || c >= n);
            even[j] = none ? (Pair16)kFar : __builtin_bit_cast(Pair16, raw[j] & 0x00ff00ffu);
            odd[j] = none ? (Pair16)kFar : __builtin_bit_cast(Pair16, (raw[j] >> 8) & 0x00ff00ffu);
        }
#pragma unroll
        for (int i = 0; i < kSeg; ++i) {
            const int c = c0 + i;
            if (c >= n) break;
            Pair16 e = even[i + kWin], f = odd[i + kWin];
#pragma unroll
            for (int d = 1; d <= kWin; ++d) {
                e = __builtin_elementwise_min(
                    e, __builtin_elementwise_min(even[i + kWin + d], even[i + kWin - d]) +
                           (Pair16)(unsigned short)(d * d));
                f = __builtin_elementwise_min(
                    f, __builtin_elementwise_min(odd[i + kWin + d], odd[i + kWin - d]) +
                           (Pair16)(unsigned short)(d * d));
            }
            int best[4] = {e.x, f.x, e.y, f.y};
            const int64_t v = base + (int64_t)c * stride;
            uint32_t p = 0x01010101u;
            if (MODE == 1) p = *reinterpret_cast<const uint32_t*>(pore + v);
            uint32_t word = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (walls)
                    best[j] = wall_min(b, walls, x0 + j, ax == 1 ? c : o, ax == 1 ? o : c, best[j]);
                if (cap > (kWin + 1) * (kWin + 1) && best[j] > (kWin + 1) * (kWin + 1))
                    best[j] = line_min_from(in, base + j, stride, c, n, per, best[j], kWin + 1);
                if (MODE == 0) {
                    word |= (uint32_t)min(best[j], cap) << (8 * j);
                } else {
                    const uint32_t near = ((p >> (8 * j)) & 0xffu) && best[j] < cap ? 1u : 0u;
                    cnt += (int)near;
                    word |= near << (8 * j);
                }
            }
            if (MODE == 0)
                *reinterpret_cast<uint32_t*>(out + v) = word;
            else if (nw)
                *reinterpret_cast<uint32_t*>(nw + v) = word;
        }
    }
    if (MODE == 1) {
        for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
        __shared__ int ws[kPrepThreads / 64];
        if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = cnt;
        __syncthreads();
        if (threadIdx.x == 0) {
            int t = 0;
            for (int i = 0; i < kPrepThreads / 64; ++i) t += ws[i];
            part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
        }
    }
}

// Fixed-order sum of n partial counts (one workgroup of kSumThreads threads).
__global__ void __launch_bounds__(kSumThreads) sum_kernel(const int* __restrict__ part,
                                                          int64_t n, long long* __restrict__ out) {
    __shared__ long long sh[kSumThreads];
    long long s = 0;
    for (int64_t i = threadIdx.x; i < n; i += kSumThreads) s += part[i];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int h = kSumThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) sh[threadIdx.x] += sh[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sh[0];
}

// ---- union-find labelling of the centres

__device__ __forceinline__ int32_t label_load(const int32_t* L, int32_t i) {
    return __hip_atomic_load(L + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of i: parents are never larger than their children, so the walk strictly decreases. On
// the way every entry passed is pointed at its grandparent (path halving), so that chains stay
// short; the store races only with stores of other ancestors and with a link that another
// thread is making of the entry, and that thread goes on to unite what the entry pointed at
// (see unite), so no connection is lost.
__device__ __forceinline__ int32_t find_root(int32_t* L, int32_t i) {
    int32_t p = label_load(L, i);
    while (p != i) {
        const int32_t g = label_load(L, p);
        if (g != p) __hip_atomic_store(L + i, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        i = p;
        p = g;
    }
    return i;
}

// Link the components of centres a and b (the larger root goes under the smaller). A failed
// link means another thread gave the root a parent first; the loop continues from there.
__device__ void unite(int32_t* L, int32_t a, int32_t b) {
    while (true) {
        a = find_root(L, a);
        b = find_root(L, b);
        if (a == b) return;
        if (a > b) {
            const int32_t t = a;
            a = b;
            b = t;
        }
        const int32_t old = atomicMin(L + b, a);
        if (old == b) return;
        b = old;
    }
}

// The labelling works on the runs of consecutive centres within a 64-voxel word of a row: a run's
// label lies at its first voxel, and no other entry is touched. A workgroup first labels a tile of
// 16 x 16 words (y by z) in LDS and writes each run's label as the tile's root, so that only runs
// that meet across a face of a tile (or the edge of a word) are united in memory, and chains there
// are short. (256^3, mean over the radii of a drainage: with every pair of runs united in memory
// the merge took 171 us, up to 750 at the widest radii, in chains of labels that other XCDs
// change, and the initial labels 8; now 17 for the tiles and 35, at most 59, for the rest.)
constexpr int kTile = 16;                        // words of a tile along y and along z
constexpr int kTileRuns = 32, kTileLd = 33;      // runs of a word at most; padded against conflicts

// Bits of the word that start a run, and the first voxel of the run of the word that holds bit x.
__device__ __forceinline__ uint64_t run_starts(uint64_t m) { return m & ~(m << 1); }
__device__ __forceinline__ int run_start(uint64_t m, int x) {
    const uint64_t gap = ~m & ((1ull << x) - 1ull);
    return gap ? 64 - __clzll((long long)gap) : 0;
}

// Labels of the runs of one tile: a run's own slot in LDS is 32 * (its word in the tile) + (its
// first bit / 2), which no two runs share and which orders as the voxels do. flag: not reached.
__global__ void __launch_bounds__(kTile * kTile) ccl_tile_kernel(Box b,
                                                                 const uint64_t* __restrict__ centre,
                                                                 int32_t* __restrict__ L,
                                                                 uint8_t* __restrict__ flag) {
    __shared__ int32_t lab[kTile * kTile * kTileLd];
    __shared__ uint64_t word[kTile * kTile];
    const int t = (int)threadIdx.x, yl = t & (kTile - 1), zl = t / kTile;
    const int nty = (b.ny + kTile - 1) / kTile;
    const int w = (int)(blockIdx.x % (unsigned)b.W), tile = (int)(blockIdx.x / (unsigned)b.W);
    const int y0 = (tile % nty) * kTile, z0 = (tile / nty) * kTile;
    const bool in = y0 + yl < b.ny && z0 + zl < b.nz;
    const uint64_t m = in ? centre[((int64_t)(z0 + zl) * b.ny + y0 + yl) * b.W + w] : 0ull;
    const uint64_t starts = run_starts(m);
    word[t] = m;
    for (uint64_t s = starts; s; s &= s - 1) {
        const int k = (__ffsll((long long)s) - 1) >> 1;
        lab[t * kTileLd + k] = t * kTileRuns + k;
    }
    __syncthreads();
    // As find_root and unite, over slots.
    auto at = [&](int v) { return lab + (v / kTileRuns) * kTileLd + (v & (kTileRuns - 1)); };
    auto load = [&](int v) {
        return __hip_atomic_load(at(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto root = [&](int v) {
        for (int p = load(v); p != v;) {
            const int g = load(p);
            if (g != p) __hip_atomic_store(at(v), g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            v = p;
            p = g;
        }
        return v;
    };
    for (int side = 0; side < 2; ++side) {
        if ((side ? zl : yl) == 0) continue;
        const int u = side ? t - kTile : t - 1;
        const uint64_t q = word[u];
        for (uint64_t f = run_starts(m & q); f; f &= f - 1) {
            const int x = __ffsll((long long)f) - 1;
            int i = t * kTileRuns + (run_start(m, x) >> 1);
            int j = u * kTileRuns + (run_start(q, x) >> 1);
            while (true) {
                i = root(i);
                j = root(j);
                if (i == j) break;
                const int hi = max(i, j), lo = min(i, j), old = atomicMin(at(hi), lo);
                if (old == hi) break;
                i = old;
                j = lo;
            }
        }
    }
    __syncthreads();
    for (uint64_t s = starts; s; s &= s - 1) {
        const int x = __ffsll((long long)s) - 1, own = t * kTileRuns + (x >> 1), r = root(own);
        // The root's first voxel: its word in the tile, and which bit of the pair starts a run.
        const int rt = r / kTileRuns, pair = 2 * (r & (kTileRuns - 1));
        const int bit = pair + ((run_starts(word[rt]) >> pair) & 1ull ? 0 : 1);
        const int64_t row = (int64_t)(z0 + zl) * b.ny + y0 + yl;
        const int64_t rr = (int64_t)(z0 + rt / kTile) * b.ny + y0 + (rt & (kTile - 1));
        L[row * b.nx + 64 * w + x] = (int32_t)(rr * b.nx + 64 * w + bit);
        if (r == own) flag[row * b.nx + 64 * w + x] = 0;
    }
}

// Unions that no tile holds: blockIdx.y 0 across the edges of words along x (and the periodic x
// face), 1 across the -y faces of the tiles, 2 across the -z faces. Two rows' runs that overlap are
// united once, at the first overlapping x: where both left neighbours are centres too, the pair to
// the left has linked the same runs, which continue across the edge of the word.
__global__ void __launch_bounds__(256) ccl_join_kernel(Box b, const uint64_t* __restrict__ centre,
                                                       int32_t* L) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int w = (int)(k % b.W);
    const int64_t line = k / b.W;
    int y, z, c;
    if (blockIdx.y == 0) {
        if (line >= (int64_t)b.ny * b.nz) return;
        const uint64_t* r = centre + line * b.W;
        if (!(r[w] & 1ull)) return;
        const int64_t base = line * b.nx;
        if (w > 0) {
            if (r[w - 1] >> 63)
                unite(L, (int32_t)(base + 64 * w),
                      (int32_t)(base + 64 * (w - 1) + run_start(r[w - 1], 63)));
        } else if ((b.per & 1) && b.nx > 1) {
            const int e = b.nx - 1;
            const uint64_t last = r[e >> 6];
            if ((last >> (e & 63)) & 1ull)
                unite(L, (int32_t)base, (int32_t)(base + 64 * (e >> 6) + run_start(last, e & 63)));
        }
        return;
    }
    if (blockIdx.y == 1) {
        const int nty = (b.ny + kTile - 1) / kTile;
        if (line >= (int64_t)nty * b.nz) return;
        y = (int)(line % nty) * kTile;
        z = (int)(line / nty);
        c = y > 0 ? y - 1 : (b.per & 2) ? b.ny - 1 : -1;
        if (c < 0 || c == y) return;
    } else {
        if (line >= (int64_t)b.ny * ((b.nz + kTile - 1) / kTile)) return;
        y = (int)(line % b.ny);
        z = (int)(line / b.ny) * kTile;
        c = z > 0 ? z - 1 : (b.per & 4) ? b.nz - 1 : -1;
        if (c < 0 || c == z) return;
    }
    const int64_t row = (int64_t)z * b.ny + y;
    const int64_t rn = blockIdx.y == 1 ? (int64_t)z * b.ny + c : (int64_t)c * b.ny + y;
    const uint64_t *r = centre + row * b.W, *q = centre + rn * b.W;
    const uint64_t o = r[w] & q[w], before = w > 0 ? (r[w - 1] & q[w - 1]) >> 63 : 0ull;
    for (uint64_t f = o & ~((o << 1) | before); f; f &= f - 1) {
        const int x = __ffsll((long long)f) - 1;
        unite(L, (int32_t)(row * b.nx + 64 * w + run_start(r[w], x)),
              (int32_t)(rn * b.nx + 64 * w + run_start(q[w], x)));
    }
}

// Flag the roots of the runs in the z = 0 plane (rows 0 .. ny-1). Every writer stores 1.
__global__ void __launch_bounds__(256) ccl_mark_kernel(Box b, const uint64_t* __restrict__ centre,
                                                       int32_t* L, uint8_t* __restrict__ flag) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= (int64_t)b.ny * b.W) return;
    const int32_t v0 = (int32_t)(k / b.W * b.nx + k % b.W * 64);
    for (uint64_t m = run_starts(centre[k]); m; m &= m - 1)
        flag[find_root(L, v0 + __ffsll((long long)m) - 1)] = 1;
}

// Reach bits: the runs whose root is flagged.
__global__ void __launch_bounds__(256) ccl_reach_kernel(Box b, const uint64_t* __restrict__ centre,
                                                        int32_t* L,
                                                        const uint8_t* __restrict__ flag,
                                                        uint64_t* __restrict__ reach) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= b.nwords) return;
    const int32_t v0 = (int32_t)(k / b.W * b.nx + k % b.W * 64);
    uint64_t out = 0;
    for (uint64_t m = centre[k]; m;) {
        const uint64_t low = m & (0ull - m), run = m & ~(m + low);   // the lowest run in the word
        if (flag[find_root(L, v0 + __ffsll((long long)low) - 1)]) out |= run;
        m &= ~run;
    }
    reach[k] = out;
}

// Largest d2 over pore voxels and the pore count: eight consecutive voxels per thread (wide
// loads; the flat arrays are 256-byte aligned), per-workgroup results, then one workgroup
// combines them.
__global__ void __launch_bounds__(kPrepThreads) pore_max_kernel(int64_t n,
                                                               const uint8_t* __restrict__ pore,
                                                               const int32_t* __restrict__ d2,
                                                               long long* __restrict__ part) {
    const int64_t v0 = 8 * ((int64_t)blockIdx.x * kPrepThreads + threadIdx.x);
    int mx = -1, cnt = 0;
    if (v0 + 8 <= n) {
        const uint32_t pm = nonzero_bytes(*reinterpret_cast<const uint64_t*>(pore + v0));
        const int4 a = *reinterpret_cast<const int4*>(d2 + v0);
        const int4 c = *reinterpret_cast<const int4*>(d2 + v0 + 4);
        const int dv[8] = {a.x, a.y, a.z, a.w, c.x, c.y, c.z, c.w};
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if ((pm >> i) & 1u) {
                mx = max(mx, dv[i]);
                ++cnt;
            }
    } else {
        for (int64_t v = v0; v < n; ++v)
            if (pore[v]) {
                mx = max(mx, d2[v]);
                ++cnt;
            }
    }
    for (int off = 32; off > 0; off >>= 1) {
        mx = max(mx, __shfl_xor(mx, off));
        cnt += __shfl_xor(cnt, off);
    }
    __shared__ int wmax[kPrepThreads / 64], wcnt[kPrepThreads / 64];
    if ((threadIdx.x & 63) == 0) {
        wmax[threadIdx.x >> 6] = mx;
        wcnt[threadIdx.x >> 6] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int m = -1, c = 0;
        for (int i = 0; i < kPrepThreads / 64; ++i) {
            m = max(m, wmax[i]);
            c += wcnt[i];
        }
        part[2 * blockIdx.x] = m;
        part[2 * blockIdx.x + 1] = c;
    }
}

// Combines nblk (max, count) pairs into out[0] (max) and out[1] (total count).
__global__ void __launch_bounds__(kSumThreads) max_count_kernel(const long long* __restrict__ part,
                                                                int64_t nblk,
                                                                long long* __restrict__ out) {
    __shared__ long long smax[kSumThreads], scnt[kSumThreads];
    long long m = -1, c = 0;
    for (int64_t i = threadIdx.x; i < nblk; i += kSumThreads) {
        m = max(m, part[2 * i]);
        c += part[2 * i + 1];
    }
    smax[threadIdx.x] = m;
    scnt[threadIdx.x] = c;
    __syncthreads();
    for (int h = kSumThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            smax[threadIdx.x] = max(smax[threadIdx.x], smax[threadIdx.x + h]);
            scnt[threadIdx.x] += scnt[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = smax[0];
        out[1] = scnt[0];
    }
}

__global__ void __launch_bounds__(256) relabel_kernel(Box b, const int32_t* __restrict__ labels,
                                                      const int8_t* __restrict__ kind,
                                                      const int32_t* __restrict__ e2,
                                                      int32_t within, int32_t new_label,
                                                      int32_t* __restrict__ out) {
    const VoxelIdx t = voxel_of(b);
    if (!t.active) return;
    const int32_t l = labels[t.v];
    out[t.v] = (kind[l] == LBM_LABEL_SOLID && e2[t.v] <= within) ? new_label : l;
}

__global__ void __launch_bounds__(256) mixing_kernel(Box b, const int32_t* __restrict__ labels,
                                                     const int8_t* __restrict__ kind, int nmix,
                                                     int32_t pore_label,
                                                     int32_t* __restrict__ out) {
    const VoxelIdx t = voxel_of(b);
    if (!t.active) return;
    const int64_t plane = (int64_t)b.nx * b.ny;
    const int z = t.row / b.ny;
    const int64_t xy = t.v - (int64_t)z * plane;
    const int32_t l = labels[t.v];
    bool open = false;
    if (kind[l] == LBM_LABEL_SOLID) {
        if (z < nmix && kind[labels[(int64_t)(b.nz - 1) * plane + xy]] != LBM_LABEL_SOLID)
            open = true;
        if (z >= b.nz - nmix && kind[labels[xy]] != LBM_LABEL_SOLID) open = true;
    }
    out[t.v] = open ? pore_label : l;
}

// ---------------------------------------------------------------------------------------------
// Host side

// Device buffers of one call; the destructor waits for the stream, then frees them. Buffers of
// kSmallBlock bytes and more are carved from one allocation, since each of that size costs its own
// mapping; smaller ones are gathered in blocks that stay below it, which the runtime serves from
// memory it holds (an allocation and its release: 1.3 us below 2 MiB, 17 and more above; 64^3, all in
// one against in small blocks: mixing layer 222 / 187 us, relabelling 267 / 231, distances 165 / 131).
struct Scratch {
    static constexpr size_t kSmallBlock = size_t(2) << 20;
    hipStream_t s;
    struct Want { void** ptr; size_t bytes; };
    std::vector<Want> wants;
    std::vector<void*> blocks;
    hipError_t err = hipSuccess;
    explicit Scratch(hipStream_t st) : s(st) {}
    ~Scratch() {
        if (!blocks.empty()) (void)hipStreamSynchronize(s);
        for (void* p : blocks) (void)hipFree(p);
    }
    // *ptr will hold `count` elements, 256-byte aligned, once get() has succeeded.
    template <typename T>
    void want(T** ptr, int64_t count) {
        wants.push_back(Want{(void**)ptr,
                             (std::max<size_t>(1, sizeof(T) * (size_t)count) + 255) / 256 * 256});
    }
    bool get() {
        for (size_t k = 0; k < wants.size();) {   // blocks of consecutive small buffers
            size_t bytes = 0, e = k;
            for (; e < wants.size(); ++e) {
                if (wants[e].bytes >= kSmallBlock) continue;
                if (bytes + wants[e].bytes >= kSmallBlock) break;
                bytes += wants[e].bytes;
            }
            if (bytes && !block(k, e, bytes, true)) return false;
            k = e;
        }
        size_t bytes = 0;
        for (const Want& w : wants) bytes += w.bytes >= kSmallBlock ? w.bytes : 0;
        return !bytes || block(0, wants.size(), bytes, false);
    }
    // One allocation of `bytes` for the small (or the other) buffers from k to e - 1.
    bool block(size_t k, size_t e, size_t bytes, bool small) {
        void* p = nullptr;
        err = hipMalloc(&p, bytes);
        if (err != hipSuccess) return false;
        blocks.push_back(p);
        size_t off = 0;
        for (; k < e; ++k)
            if ((wants[k].bytes < kSmallBlock) == small) {
                *wants[k].ptr = (char*)p + off;
                off += wants[k].bytes;
            }
        return true;
    }
    // Status for a failed allocation: out of memory, or no usable device.
    lbm_status failed(const char* what) const {
        if (err == hipErrorOutOfMemory)
            return fail(LBM_ERR_OOM, std::string("no device memory for ") + what);
        return fail(LBM_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(err));
    }
};

lbm_status check_box(int32_t nx, int32_t ny, int32_t nz, const int32_t* periodic, Box* b) {
    if (nx < 1 || ny < 1 || nz < 1 || nx > kMaxDim || ny > kMaxDim || nz > kMaxDim)
        return fail(LBM_ERR_ARG, "image sizes must lie in [1, 16384]");
    const int64_t nvox = (int64_t)nx * ny * nz;
    if (nvox >= (int64_t)1 << 31) return fail(LBM_ERR_ARG, "nx*ny*nz must be below 2^31");
    b->nx = nx;
    b->ny = ny;
    b->nz = nz;
    b->W = (nx + 63) / 64;
    b->nvox = nvox;
    b->nwords = (int64_t)ny * nz * b->W;
    b->per = 0;
    if (periodic)
        for (int a = 0; a < 3; ++a)
            if (periodic[a]) b->per |= 1 << a;
    b->tpb = std::min(kPrepThreads, 64 * b->W);
    b->chunks = (nx + b->tpb - 1) / b->tpb;
    return LBM_OK;
}

// Grid of the per-voxel kernels (one workgroup per row and chunk of x) and of the bit packing.
dim3 vox_grid(const Box& b) { return dim3((unsigned)(b.ny * b.nz), (unsigned)b.chunks); }
// Row pass: four voxels per thread, 1 << row_shift threads per row.
int row_shift(const Box& b) {
    int s = 0;
    while (s < 8 && (4 << s) < b.nx) ++s;
    return s;
}
dim3 row_grid(const Box& b) {
    const int s = row_shift(b), rows = 256 >> s, span = 4 << s;
    return dim3((unsigned)((b.ny * b.nz + rows - 1) / rows), (unsigned)((b.nx + span - 1) / span));
}
dim3 pack8_grid(const Box& b) { return dim3((unsigned)((b.nwords + 31) / 32)); }
dim3 pack_grid(const Box& b) {
    const int64_t per_block = 4 * kWordsPerWave;   // four waves of kWordsPerWave words
    return dim3((unsigned)((b.nwords + per_block - 1) / per_block));
}

lbm_status check_labels(const Box& b, const int32_t* labels, int32_t n_labels,
                        const int8_t* kind) {
    if (!labels || !kind || n_labels < 1) return fail(LBM_ERR_ARG, "labels and kinds are required");
    for (int32_t l = 0; l < n_labels; ++l)
        if (kind[l] < LBM_LABEL_SOLID || kind[l] > LBM_LABEL_PORE_INIT)
            return fail(LBM_ERR_ARG, "label_kind[" + std::to_string(l) +
                                         "] is not a lbm_label_kind");
    for (int64_t v = 0; v < b.nvox; ++v)
        if (labels[v] < 0 || labels[v] >= n_labels)
            return fail(LBM_ERR_ARG, "labels[" + std::to_string(v) + "] is outside [0, n_labels)");
    return LBM_OK;
}

// Packs a predicate into row bits, with the wide kernel when rows are a multiple of 8 long.
template <typename P, typename P8>
lbm_status pack(const Box& b, P pred, P8 pred8, uint64_t* bits, hipStream_t s) {
    if ((b.nx & 7) == 0)
        hipLaunchKernelGGL(pack8_kernel<P8>, pack8_grid(b), dim3(256), 0, s, b, pred8, bits);
    else
        hipLaunchKernelGGL(pack_kernel<P>, pack_grid(b), dim3(256), 0, s, b, pred, bits);
    HIP_TRY(hipGetLastError());
    return LBM_OK;
}

// Row search limit: the largest distance along x that can still be below the cap.
int row_limit(const Box& b, int32_t cap) {
    int lim = (b.per & 1) ? b.nx / 2 : b.nx - 1;
    if (cap < kInf) lim = (int)std::min<int64_t>(lim, (int64_t)std::sqrt((double)cap) + 1);
    return lim;
}

// Grid of the line passes along axis ax: one workgroup per (line group, segment, chunk of x).
dim3 seg_grid(const Box& b, int ax) {
    const int n = ax == 1 ? b.ny : b.nz, other = ax == 1 ? b.nz : b.ny;
    return dim3((unsigned)(other * ((n + kSeg - 1) / kSeg)), (unsigned)b.chunks);
}
int64_t seg_blocks(const Box& b, int ax) {
    const dim3 g = seg_grid(b, ax);
    return (int64_t)g.x * g.y;
}

// Grid of the line passes on bytes.
dim3 seg8_grid(const Box& b, int ax) {
    const int n = ax == 1 ? b.ny : b.nz, other = ax == 1 ? b.nz : b.ny;
    const int64_t segs = (int64_t)other * ((n + kSeg - 1) / kSeg);
    const int s = row_shift(b), per = 256 >> s, span = 4 << s;
    return dim3((unsigned)((segs + per - 1) / per), (unsigned)((b.nx + span - 1) / span));
}

// Fewest voxels for which a thread of a pass on bytes takes four lines: below, too few waves are left
// (512 at 2^20 voxels) to hide the longer thread, and each line has a thread of its own
// (edt_seg_kernel). us a drainage of a rock, one line / four: 32^3 318 / 352, 64^3 403 / 440, 80^3
// 441 / 462, 96^3 503 / 506, 112^3 599 / 598, 128^3 681 / 680, 160^3 1102 / 1047; a growth in 48^3
// 124 / 135, 100^3 144 / 151, 128^3 160 / 152.
constexpr int64_t kQuadVoxels = int64_t(1) << 20;

// One line pass in MODE 0 or 1 (see edt_seg_kernel); *blocks receives the workgroups of the
// launch, one partial count each in MODE 1.
template <int MODE, typename T>
lbm_status line_pass(const Box& b, int ax, int32_t cap, int walls, const T* in, T* out,
                     const uint8_t* pore, uint8_t* nw, int* part, int64_t* blocks,
                     hipStream_t s) {
    if constexpr (sizeof(T) == 1) {
        if ((b.nx & 3) == 0 && b.nvox >= kQuadVoxels) {
            const dim3 g = seg8_grid(b, ax);
            hipLaunchKernelGGL((edt_seg8_kernel<MODE>), g, dim3(256), 0, s, b, ax, row_shift(b),
                               cap, walls, in, out, pore, nw, part);
            HIP_TRY(hipGetLastError());
            if (blocks) *blocks = (int64_t)g.x * g.y;
            return LBM_OK;
        }
    }
    // MODE 1: kPrepThreads per workgroup (its block sum needs them all): whenever b.tpb is
    // smaller, there is one chunk per row, which 256 threads cover as well.
    const dim3 g = seg_grid(b, ax);
    hipLaunchKernelGGL((edt_seg_kernel<MODE, T>), g, dim3(MODE == 1 ? kPrepThreads : b.tpb), 0, s,
                       b, ax, cap, walls, in, out, pore, nw, part);
    HIP_TRY(hipGetLastError());
    if (blocks) *blocks = (int64_t)g.x * g.y;
    return LBM_OK;
}

// Row and y passes in one (see edt_plane_kernel).
template <bool BYTES>
lbm_status edt_plane(const Box& b, const uint64_t* bits, const uint8_t* image, int32_t cap,
                     int32_t* mid, hipStream_t s) {
    const int chunks = (b.nx + kPlaneCols - 1) / kPlaneCols;
    const size_t lds = sizeof(int32_t) * kPlaneLd * (size_t)plane_rows(b) +
                       (BYTES ? sizeof(uint64_t) * (size_t)b.ny * b.W : 0);
    hipLaunchKernelGGL(edt_plane_kernel<BYTES>, dim3((unsigned)((int64_t)b.nz * chunks)),
                       dim3(kPlaneThreads), lds, s, b, bits, image, row_limit(b, cap), cap, mid);
    HIP_TRY(hipGetLastError());
    return LBM_OK;
}

// Row and y passes of the transform of the feature bits: leaves the y-pass result in mid
// (row-pass scratch in tmp). T holds values up to cap (int32_t, or uint8_t for caps <= 255).
template <typename T>
lbm_status edt_xy(const Box& b, const uint64_t* bits, int32_t cap, T* tmp, T* mid,
                  hipStream_t s) {
    if constexpr (sizeof(T) == 4)
        if (plane_pass(b)) return edt_plane<false>(b, bits, nullptr, cap, mid, s);
    const bool flat = b.ny == 1;   // no line along y: the row pass is both
    hipLaunchKernelGGL(edt_row_kernel<T>, row_grid(b), dim3(256), 0, s, b, bits,
                       row_shift(b), row_limit(b, cap), cap, flat ? mid : tmp);
    HIP_TRY(hipGetLastError());
    if (flat) return LBM_OK;
    return line_pass<0, T>(b, 1, cap, 0, tmp, mid, nullptr, nullptr, nullptr, nullptr, s);
}

// Full squared distance transform of the feature bits into out (tmp: a second buffer of nvox);
// values at or above cap are clipped to cap.
template <typename T>
lbm_status edt(const Box& b, const uint64_t* bits, int32_t cap, int walls, T* tmp, T* out,
               hipStream_t s) {
    if (lbm_status st = edt_xy<T>(b, bits, cap, out, tmp, s)) return st;
    return line_pass<0, T>(b, 2, cap, walls, tmp, out, nullptr, nullptr, nullptr, nullptr, s);
}

// The transform of a byte image, without a cap; -1 stands for no feature. bits: scratch for the
// row words, tmp: for nvox distances.
lbm_status edt_image(const Box& b, const uint8_t* image, uint64_t* bits, int walls, int32_t* tmp,
                     int32_t* out, hipStream_t s) {
    // Wide packing reads 8 voxels per 8-byte load: rows of whole bytes and an aligned image.
    const bool wide = (b.nx & 7) == 0 && ((uintptr_t)image & 7) == 0;
    if (wide && b.nx <= kPlaneBytes && plane_pass(b)) {
        if (lbm_status st = edt_plane<true>(b, nullptr, image, kInf, tmp, s)) return st;
    } else {
        if (wide)
            hipLaunchKernelGGL(pack8_kernel<Wide8Nonzero>, pack8_grid(b), dim3(256), 0, s, b,
                               Wide8Nonzero{image}, bits);
        else
            hipLaunchKernelGGL(pack_kernel<FeatureNonzero>, pack_grid(b), dim3(256), 0, s, b,
                               FeatureNonzero{image}, bits);
        HIP_TRY(hipGetLastError());
        if (lbm_status st = edt_xy<int32_t>(b, bits, kInf, out, tmp, s)) return st;
    }
    hipLaunchKernelGGL((edt_seg_kernel<2, int32_t>), seg_grid(b, 2), dim3(b.tpb), 0, s, b, 2, kInf,
                       walls, (const int32_t*)tmp, out, nullptr, nullptr, nullptr);
    HIP_TRY(hipGetLastError());
    return LBM_OK;
}

struct DrainBuffers {
    uint8_t* pore;
    int32_t* d2;      // squared distance to the solid
    int32_t* tmp;     // transform scratch
    int32_t* mid;     // transform scratch
    int32_t* label;   // union-find labels
    uint8_t* flag;    // roots that touch the inlet plane
    uint64_t* centre;
    uint64_t* reach;
    int* part;        // per-workgroup counts
    long long* part2; // final sums: count, or (max, count)
    long long* pairs; // (max, count) per workgroup of the pore reduction
};

// Reach bits: the centres whose face-connected component touches the z = 0 plane.
lbm_status connect_to_inlet(const Box& b, const DrainBuffers& db, hipStream_t s) {
    const unsigned blocks = (unsigned)((b.nwords + 255) / 256);
    const uint64_t* centre = db.centre;
    const int64_t nty = (b.ny + kTile - 1) / kTile, ntz = (b.nz + kTile - 1) / kTile;
    hipLaunchKernelGGL(ccl_tile_kernel, dim3((unsigned)(nty * ntz * b.W)), dim3(kTile * kTile), 0, s,
                       b, centre, db.label, db.flag);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(ccl_join_kernel, dim3(blocks, 3), dim3(256), 0, s, b, centre, db.label);
    HIP_TRY(hipGetLastError());
    const int64_t plane = (int64_t)b.ny * b.W;
    hipLaunchKernelGGL(ccl_mark_kernel, dim3((unsigned)((plane + 255) / 256)), dim3(256), 0, s, b,
                       centre, db.label, db.flag);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(ccl_reach_kernel, dim3(blocks), dim3(256), 0, s, b, centre, db.label,
                       (const uint8_t*)db.flag, db.reach);
    HIP_TRY(hipGetLastError());
    return LBM_OK;
}

// The passes of a drainage dilation: the number of pore voxels closer than sqrt(k) to a feature
// bit, into db.part2, and their mask when nw_dev is not null.
template <typename T>
lbm_status dilate_count(const Box& b, const uint64_t* feat, int32_t k, T* tmp, T* mid,
                        const DrainBuffers& db, uint8_t* nw_dev, hipStream_t s) {
    if (lbm_status st = edt_xy<T>(b, feat, k, tmp, mid, s)) return st;
    int64_t blocks = 0;
    if (lbm_status st = line_pass<1, T>(b, 2, k, 0, mid, nullptr, db.pore, nw_dev, db.part,
                                        &blocks, s))
        return st;
    hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(kSumThreads), 0, s, (const int*)db.part, blocks,
                       db.part2);
    HIP_TRY(hipGetLastError());
    return LBM_OK;
}

// Non-wetting count for squared radius k; writes the mask to nw_dev when it is not null.
lbm_status drain_eval(const Box& b, const DrainBuffers& db, int32_t k, bool inlet,
                      uint8_t* nw_dev, int64_t* n_nw, hipStream_t s) {
    FeatureCentre fc{db.pore, db.d2, k};
    if (lbm_status st = pack(b, fc, Wide8Centre{db.pore, db.d2, k}, db.centre, s)) return st;
    const uint64_t* feat = db.centre;
    if (inlet) {
        if (lbm_status st = connect_to_inlet(b, db, s)) return st;
        feat = db.reach;
    }
    // The passes hold values up to k: bytes while they suffice (k <= 255, spheres of a radius up
    // to 15 voxels, all that a rock's pores admit), a quarter of the int32 traffic.
    if (k <= 255) {
        if (lbm_status st = dilate_count(b, feat, k, (uint8_t*)db.tmp, (uint8_t*)db.mid, db, nw_dev, s))
            return st;
    } else if (lbm_status st = dilate_count(b, feat, k, db.tmp, db.mid, db, nw_dev, s)) {
        return st;
    }
    long long h = 0;
    HIP_TRY(hipMemcpyAsync(&h, db.part2, sizeof h, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    *n_nw = h;
    return LBM_OK;
}

// ---- Scratch of the allocation-free distance transform -------------------------------------
// lbm_prep_distance_noalloc keeps its work buffers (row words, one int32 transform pass) in this
// file-scope device array: one copy per GPU, held until the process ends, shared by every call on
// that GPU. Host code never passes the array's name to a kernel: its device address is taken once
// per device with hipGetSymbolAddress, with that device current.
constexpr size_t kNoAllocScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char noalloc_scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[kMaxDevices] = {};

// Device address of the current device's scratch array.
lbm_status noalloc_scratch_of_current_device(void** out) {
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(LBM_ERR_DEVICE, "device index out of range");
    std::lock_guard<std::mutex> lock(g_noalloc_mu);
    if (!g_noalloc_ptr[dev]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(noalloc_scratch));
        if (e != hipSuccess || !ptr)
            return fail(LBM_ERR_DEVICE, std::string("scratch address: ") + hipGetErrorString(e));
        g_noalloc_ptr[dev] = ptr;
    }
    *out = g_noalloc_ptr[dev];
    return LBM_OK;
}

}  // namespace

namespace lbm {

lbm_status morph_distance(int nx, int ny, int nz, int periodic, const uint64_t* label_bits,
                          uint64_t* other_bits, int32_t cap, uint8_t* tmp, uint8_t* to_a,
                          uint8_t* to_other, hipStream_t s) {
    if (cap < 1 || cap > 255) return fail(LBM_ERR_ARG, "internal: distance cap outside [1, 255]");
    const int32_t per[3] = {periodic & 1, (periodic >> 1) & 1, (periodic >> 2) & 1};
    Box b{};
    if (lbm_status st = check_box(nx, ny, nz, per, &b)) return st;
    if (lbm_status st = edt<uint8_t>(b, label_bits, cap, 0, tmp, to_a, s)) return st;
    hipLaunchKernelGGL(invert_bits_kernel, dim3((unsigned)((b.nwords + 255) / 256)), dim3(256), 0,
                       s, b, label_bits, other_bits);
    HIP_TRY(hipGetLastError());
    return edt<uint8_t>(b, other_bits, cap, 7, tmp, to_other, s);
}

}  // namespace lbm

lbm_status lbm_prep_distance(int32_t nx, int32_t ny, int32_t nz, const int32_t periodic[3],
                             int32_t wall_axes, const uint8_t* feature, int32_t* dist_sq,
                             void* hip_stream) {
    clear_error();
    Box b{};
    if (lbm_status st = check_box(nx, ny, nz, periodic, &b)) return st;
    if (!feature || !dist_sq) return fail(LBM_ERR_ARG, "null argument");
    if (wall_axes < 0 || wall_axes > 7) return fail(LBM_ERR_ARG, "wall_axes must lie in [0, 7]");
    hipStream_t s = (hipStream_t)hip_stream;
    Scratch sc(s);
    uint8_t* f;
    uint64_t* bits;
    int32_t *tmp, *out;
    sc.want(&f, b.nvox);
    sc.want(&bits, b.nwords);
    sc.want(&tmp, b.nvox);
    sc.want(&out, b.nvox);
    if (!sc.get()) return sc.failed("the transform");
    HIP_TRY(copy_to_device(f, feature, (size_t)b.nvox, s));
    if (lbm_status st = edt_image(b, f, bits, wall_axes, tmp, out, s)) return st;
    HIP_TRY(copy_to_host(dist_sq, out, sizeof(int32_t) * (size_t)b.nvox, s));
    return LBM_OK;
}

lbm_status lbm_prep_distance_noalloc(int32_t nx, int32_t ny, int32_t nz, const int32_t periodic[3],
                                     int32_t wall_axes, const uint8_t* feature_dev,
                                     int32_t* dist_sq_dev, void* hip_stream) {
    clear_error();
    Box b{};
    if (lbm_status st = check_box(nx, ny, nz, periodic, &b)) return st;
    if (!feature_dev || !dist_sq_dev) return fail(LBM_ERR_ARG, "null argument");
    if (wall_axes < 0 || wall_axes > 7) return fail(LBM_ERR_ARG, "wall_axes must lie in [0, 7]");
    if (((uintptr_t)dist_sq_dev & 3) != 0)
        return fail(LBM_ERR_ARG, "dist_sq_dev must be 4-byte aligned");
    const size_t words_bytes = ((size_t)8 * (size_t)b.nwords + 255) / 256 * 256;
    const size_t need = words_bytes + sizeof(int32_t) * (size_t)b.nvox;
    if (need > kNoAllocScratchBytes)
        return fail(LBM_ERR_ARG, "image too large for the allocation-free transform: it needs " +
                                     std::to_string(need) + " bytes of scratch (8 per 64-voxel "
                                     "row word + 4 per voxel), the limit is " +
                                     std::to_string(kNoAllocScratchBytes));
    void* base = nullptr;
    if (lbm_status st = noalloc_scratch_of_current_device(&base)) return st;
    uint64_t* bits = (uint64_t*)base;
    int32_t* tmp = (int32_t*)((char*)base + words_bytes);
    hipStream_t s = (hipStream_t)hip_stream;
    return edt_image(b, feature_dev, bits, wall_axes, tmp, dist_sq_dev, s);
}

lbm_status lbm_prep_drain(int32_t nx, int32_t ny, int32_t nz, const int32_t periodic[3],
                          const uint8_t* pore, const lbm_drain_params* dp, uint8_t* nw,
                          lbm_drain_result* out, void* hip_stream) {
    clear_error();
    Box b{};
    if (lbm_status st = check_box(nx, ny, nz, periodic, &b)) return st;
    if (!pore || !dp || !nw || !out) return fail(LBM_ERR_ARG, "null argument");
    if (!(dp->target_sw >= 0.0 && dp->target_sw < 1.0))
        return fail(LBM_ERR_ARG, "target_sw must lie in [0, 1)");
    if (dp->inlet != 0 && dp->inlet != 1) return fail(LBM_ERR_ARG, "inlet must be 0 or 1");
    const bool inlet = dp->inlet == 1;
    if (inlet && (b.per & 4)) return fail(LBM_ERR_ARG, "an inlet needs a non-periodic z axis");
    hipStream_t s = (hipStream_t)hip_stream;
    Scratch sc(s);
    DrainBuffers db{};
    uint8_t* nw_dev;
    sc.want(&db.pore, b.nvox);
    sc.want(&db.d2, b.nvox);
    sc.want(&db.tmp, b.nvox);
    sc.want(&db.mid, b.nvox);
    sc.want(&db.centre, b.nwords);
    sc.want(&db.part, seg_blocks(b, 2));   // no line pass on bytes has more workgroups
    sc.want(&db.part2, 2);
    sc.want(&db.pairs, 2 * ((b.nvox + 8 * kPrepThreads - 1) / (8 * kPrepThreads)));
    sc.want(&nw_dev, b.nvox);
    if (inlet) sc.want(&db.reach, b.nwords);
    if (!sc.get()) return sc.failed("the drainage");
    // The labelling is done before the passes of a radius begin: it uses their buffers.
    db.label = db.mid;
    db.flag = (uint8_t*)db.tmp;
    HIP_TRY(copy_to_device(db.pore, pore, (size_t)b.nvox, s));

    // D^2: distance to the solid and to the wall planes of the non-periodic faces.
    if (lbm_status st = pack(b, FeatureZero{db.pore}, Wide8Zero{db.pore}, db.centre, s))
        return st;
    const int walls = inlet ? 3 : 7;
    if (lbm_status st = edt(b, db.centre, kInf, walls, db.tmp, db.d2, s)) return st;
    const int64_t nblk = (b.nvox + 8 * kPrepThreads - 1) / (8 * kPrepThreads);
    hipLaunchKernelGGL(pore_max_kernel, dim3((unsigned)nblk), dim3(kPrepThreads), 0, s, b.nvox,
                       (const uint8_t*)db.pore, (const int32_t*)db.d2, db.pairs);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(max_count_kernel, dim3(1), dim3(kSumThreads), 0, s,
                       (const long long*)db.pairs, nblk, db.part2);
    HIP_TRY(hipGetLastError());
    long long h[2] = {0, 0};
    HIP_TRY(hipMemcpyAsync(h, db.part2, sizeof h, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    const long long kmax = h[0], npore = h[1];
    if (npore == 0) return fail(LBM_ERR_ARG, "the image has no pore voxel");
    if (kmax >= kInf) return fail(LBM_ERR_ARG, "no solid voxel and no wall: distances are unbounded");

    // Bisection for the largest k whose water saturation is at or below the target.
    lbm_drain_result r{};
    r.max_radius_sq = (int32_t)kmax;
    r.n_pore = npore;
    auto sw_of = [&](int64_t n_nw) { return 1.0 - (double)n_nw / (double)npore; };
    int32_t lo = 0, hi = (int32_t)kmax + 1;
    while (hi - lo > 1) {
        const int32_t mid = lo + (hi - lo) / 2;
        int64_t c = 0;
        if (lbm_status st = drain_eval(b, db, mid, inlet, nullptr, &c, s)) return st;
        ++r.evaluations;
        if (sw_of(c) <= dp->target_sw)
            lo = mid;
        else
            hi = mid;
    }
    r.radius_sq = std::max(lo, 1);
    if (lbm_status st = drain_eval(b, db, r.radius_sq, inlet, nw_dev, &r.n_nw, s)) return st;
    ++r.evaluations;
    r.sw = sw_of(r.n_nw);
    HIP_TRY(copy_to_host(nw, nw_dev, (size_t)b.nvox, s));
    *out = r;
    return LBM_OK;
}

lbm_status lbm_prep_relabel(int32_t nx, int32_t ny, int32_t nz, const int32_t periodic[3],
                            const int32_t* labels, int32_t n_labels, const int8_t* label_kind,
                            const uint8_t* nw, double dist, int32_t new_label,
                            int32_t* labels_out, void* hip_stream) {
    clear_error();
    Box b{};
    if (lbm_status st = check_box(nx, ny, nz, periodic, &b)) return st;
    if (!nw || !labels_out) return fail(LBM_ERR_ARG, "null argument");
    if (!(dist >= 0.0 && dist <= (double)kMaxDim)) return fail(LBM_ERR_ARG, "dist must lie in [0, 16384]");
    if (new_label < 0) return fail(LBM_ERR_ARG, "new_label must be >= 0");
    if (lbm_status st = check_labels(b, labels, n_labels, label_kind)) return st;
    // Squared distances at most dist^2 (integers): within = floor(dist^2), cap one above.
    const int32_t within = (int32_t)std::floor(dist * dist);
    const int32_t cap = within + 1;
    hipStream_t s = (hipStream_t)hip_stream;
    Scratch sc(s);
    int32_t *lab, *res, *e2, *tmp;
    int8_t* kind;
    uint8_t* m;
    uint64_t* bits;
    sc.want(&lab, b.nvox);
    sc.want(&res, b.nvox);
    sc.want(&kind, n_labels);
    sc.want(&m, b.nvox);
    sc.want(&bits, b.nwords);
    sc.want(&e2, b.nvox);
    sc.want(&tmp, b.nvox);
    if (!sc.get()) return sc.failed("the relabelling");
    HIP_TRY(copy_to_device(lab, labels, sizeof(int32_t) * (size_t)b.nvox, s));
    HIP_TRY(hipMemcpyAsync(kind, label_kind, (size_t)n_labels, hipMemcpyHostToDevice, s));
    HIP_TRY(copy_to_device(m, nw, (size_t)b.nvox, s));
    if (lbm_status st = pack(b, FeatureNonzero{m}, Wide8Nonzero{m}, bits, s)) return st;
    if (lbm_status st = edt(b, bits, cap, 0, tmp, e2, s)) return st;
    hipLaunchKernelGGL(relabel_kernel, vox_grid(b), dim3(b.tpb), 0, s, b, (const int32_t*)lab,
                       (const int8_t*)kind, (const int32_t*)e2, within, new_label, res);
    HIP_TRY(hipGetLastError());
    HIP_TRY(copy_to_host(labels_out, res, sizeof(int32_t) * (size_t)b.nvox, s));
    return LBM_OK;
}

lbm_status lbm_prep_mixing_layer(int32_t nx, int32_t ny, int32_t nz, const int32_t* labels,
                                 int32_t n_labels, const int8_t* label_kind, int32_t nmix,
                                 int32_t pore_label, int32_t* labels_out, void* hip_stream) {
    clear_error();
    Box b{};
    if (lbm_status st = check_box(nx, ny, nz, nullptr, &b)) return st;
    if (!labels_out) return fail(LBM_ERR_ARG, "null argument");
    if (nmix < 0 || nmix > nz) return fail(LBM_ERR_ARG, "nmix must lie in [0, nz]");
    if (lbm_status st = check_labels(b, labels, n_labels, label_kind)) return st;
    if (pore_label < 0 || pore_label >= n_labels || label_kind[pore_label] == LBM_LABEL_SOLID)
        return fail(LBM_ERR_ARG, "pore_label must be a pore label of the table");
    hipStream_t s = (hipStream_t)hip_stream;
    Scratch sc(s);
    int32_t *lab, *res;
    int8_t* kind;
    sc.want(&lab, b.nvox);
    sc.want(&res, b.nvox);
    sc.want(&kind, n_labels);
    if (!sc.get()) return sc.failed("the mixing layer");
    HIP_TRY(copy_to_device(lab, labels, sizeof(int32_t) * (size_t)b.nvox, s));
    HIP_TRY(hipMemcpyAsync(kind, label_kind, (size_t)n_labels, hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(mixing_kernel, vox_grid(b), dim3(b.tpb), 0, s, b, (const int32_t*)lab,
                       (const int8_t*)kind, nmix, pore_label, res);
    HIP_TRY(hipGetLastError());
    HIP_TRY(copy_to_host(labels_out, res, sizeof(int32_t) * (size_t)b.nvox, s));
    return LBM_OK;
}
