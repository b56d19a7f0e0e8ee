// HIP kernels of the surfel Gauss-Newton path for gfx950 (CDNA4).
//
// Paper: "Dense monocular SLAM by direct surfel optimization" (Trabes,
// Dondo Gazzano, Sosa Paez), Proposed Approach section, Eq. 1-10.
//
// Kernels
//   stage_kernel   table upload: descriptors copied from pinned host memory,
//                  per-frame constants H = K R K^-1 and K t (Eq. 6) formed in
//                  double; clears the work queues.
//   init_kernel    neighbour-plane initialisation (Surfel Initialization).
//   gn_kernel      the fused Gauss-Newton iterations.  A work item is a set
//                  of surfel groups inside one aligned 16 x 16-pixel block;
//                  a group fills the 64 lanes of a wavefront with pixels (four,
//                  eight or sixteen 4x4 surfels, one 8x8 or one 16x16).  Each
//                  lane loops over the neighbour frames for its pixels, with the per-pixel
//                  inverse-depth Jacobian hoisted out of the frame loop (the
//                  paper notes it does not depend on the frame); the normal
//                  equations are reduced across the surfel's lanes with DPP,
//                  and one owner lane per surfel solves its 3x3 system, all
//                  groups of the item at once.  All iterations run inside the
//                  kernel: surfels never read each other during the
//                  optimisation.  Compiled in several forms, picked by the
//                  number of work items; gn_shared_kernel is the form of
//                  large undamped grids.
//   disc_*         disc surfels (Eq. 4): Gauss-Newton, depth-buffered render,
//                  search, placement and transfer.
//   render_kernel  per-pixel inverse depth (and owning surfel) by Eq. 3.
//   regrid_*       surfel reference-frame change (Eq. 10) and re-gridding
//                  into another keyframe's tiles.
//   quantize_kernel  f32 images to f16 / u8 storage.
//
// Numerics.  The warp uses the closed form of Eq. 6 for a plane:
//   q = H u~ + (K t) id_u,   u_p = (q_x / q_z, q_y / q_z),
// which is K (R X + t) scaled by id_u.  id_u is formed in difference form
//   sigma = n . (r_u - r_s) / (n . r_s),   id_u = id_s (1 + sigma),
// equal to Eq. 3 without its cancellation.  The image gradient is the exact
// derivative of the bilinear interpolant.  Accumulation is in float, in a
// fixed order per surfel (frames in order per lane, then a fixed DPP tree),
// so a surfel's result depends neither on where it sits in a batch nor on
// the launch plan.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "sgn_internal.h"
#include "surfgn.h"

namespace sgn {

// ---------------------------------------------------------------- helpers --

// Pointers into the constant address space: the descriptor tables are not
// written while a kernel runs, so uniform reads become scalar loads.
template <class T>
using carg = const T __attribute__((address_space(4)));
template <class T>
using cptr = carg<T>*;
// Global-address-space pointers (global_load with a scalar base).
template <class T>
using gptr = const T __attribute__((address_space(1)))*;
template <class T>
using gmut = T __attribute__((address_space(1)))*;

template <typename T>
__device__ __forceinline__ float ldg(gptr<T> p);
template <>
__device__ __forceinline__ float ldg<float>(gptr<float> p) { return *p; }
template <>
__device__ __forceinline__ float ldg<_Float16>(gptr<_Float16> p) { return (float)*p; }
template <>
__device__ __forceinline__ float ldg<uint8_t>(gptr<uint8_t> p) { return (float)*p; }

template <typename T>
__device__ __forceinline__ float ldpix(const T* p);
template <>
__device__ __forceinline__ float ldpix<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float ldpix<_Float16>(const _Float16* p) { return (float)*p; }
template <>
__device__ __forceinline__ float ldpix<uint8_t>(const uint8_t* p) { return (float)*p; }

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int x) {
    return __builtin_amdgcn_mov_dpp(x, CTRL, 0xF, 0xF, true);
}

// Sum over a surfel's lanes: 4 lanes (a quad), 8 (half a DPP row), 16 (one
// row), 32 (two rows) or the whole wavefront.  Every lane of the surfel ends with the
// bitwise-same value: each step adds a lane's value and its partner's, and
// float addition is commutative.
template <int LANES>
__device__ __forceinline__ float group_sum(float x) {
#pragma clang fp contract(off)
    static_assert(LANES == 4 || LANES == 8 || LANES == 16 || LANES == 32 || LANES == 64,
                  "lanes per surfel");
    x += dpp_f<0xB1>(x);
    x += dpp_f<0x4E>(x);
    if constexpr (LANES >= 8) x += dpp_f<0x141>(x);
    if constexpr (LANES >= 16) x += dpp_f<0x140>(x);
    if constexpr (LANES >= 32) x += __shfl_xor(x, 16);
    if constexpr (LANES == 64) x += __shfl_xor(x, 32);
    return x;
}
template <int LANES>
__device__ __forceinline__ int group_sum(int x) {
    static_assert(LANES == 4 || LANES == 8 || LANES == 16 || LANES == 32 || LANES == 64,
                  "lanes per surfel");
    x += dpp_i<0xB1>(x);
    x += dpp_i<0x4E>(x);
    if constexpr (LANES >= 8) x += dpp_i<0x141>(x);
    if constexpr (LANES >= 16) x += dpp_i<0x140>(x);
    if constexpr (LANES >= 32) x += __shfl_xor(x, 16);
    if constexpr (LANES == 64) x += __shfl_xor(x, 32);
    return x;
}

// Sums of two values over a surfel's lanes at once: lane 0 of the surfel
// ends with the sum of `ev`, lane 1 with the sum of `od`.  The first
// butterfly step trades halves with the neighbour lane (each lane keeps the
// value it will own and sends the other), so the remaining steps carry one
// value instead of two; they pair lanes of equal parity only (quad_perm,
// then row rotations by 4 and 8; an 8-lane surfel instead shifts its second
// quad's sums down by 4 lanes, since a rotation would bring in the
// neighbouring surfel's).  Lanes 0 and 1 form their sums in a fixed order
// that depends only on the surfel's pixels.
template <int LANES>
__device__ __forceinline__ float pair_sum(float ev, float od, bool odd) {
#pragma clang fp contract(off)
    static_assert(LANES == 4 || LANES == 8 || LANES == 16 || LANES == 32 || LANES == 64,
                  "lanes per surfel");
    const float keep = odd ? od : ev;
    const float send = odd ? ev : od;
    float x = keep + dpp_f<0xB1>(send);   // quad_perm [1,0,3,2]
    x += dpp_f<0x4E>(x);                  // quad_perm [2,3,0,1]
    if constexpr (LANES == 4) {
    } else if constexpr (LANES == 8) {
        x += dpp_f<0x104>(x);             // row_shl:4 (lane i takes lane i + 4)
    } else {
        x += dpp_f<0x124>(x);             // row_ror:4
        x += dpp_f<0x128>(x);             // row_ror:8
    }
    if constexpr (LANES >= 32) x += __shfl_xor(x, 16);
    if constexpr (LANES == 64) x += __shfl_xor(x, 32);
    return x;
}

__device__ __forceinline__ float rcp_fast(float x) { return __builtin_amdgcn_rcpf(x); }

__device__ __forceinline__ int find_kf(cptr<KfDev> kfs, int n_kf, int item, int hint) {
    const cptr<KfDev> h = kfs + hint;
    if (item >= h->item_base && item < h->item_base + h->n_items) return hint;
    int lo = 0, hi = n_kf - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (kfs[mid].item_base <= item) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Next work item of a persistent wavefront: take one from queue q, moving on
// to the next queue when q is exhausted; `total` when every queue is empty.
__device__ __forceinline__ int pull_item(cptr<BatchHeader> hdr, uint32_t* counters,
                                         int& q, int& q_left, int lane, int total) {
    while (q_left > 0) {
        // (A plain read of the head in front of the atomic, to spare the
        // atomics on queues that are empty, doubles the trip to memory that
        // every item waits for: with 28 wavefronts per CU 16 mixed keyframes
        // in groups of four surfels took 6.4 ms against 1.6.)
        int got = 0;
        if (lane == 0) got = (int)atomicAdd(&counters[q], 1u);
        got = __builtin_amdgcn_readfirstlane(got);
        const int it = hdr->queues[q].begin + got;
        if (it < hdr->queues[q].end) return it;
        q = (q + 1 == hdr->n_queues) ? 0 : q + 1;
        --q_left;
    }
    return total;
}

// ------------------------------------------------------------ stage kernel --

// The call's table from pinned host memory to the device table, 16 bytes per
// thread, one thread per neighbour frame forming its constants, and the
// work-queue heads cleared.  A few hundred KB at most: bound by the latency
// of one read over the host link.  A copy command (on the DMA engine for the
// larger tables) and a kernel for the constants after it took 40 us from the
// copy's start to the first working kernel of a 64-keyframe update, this
// launch 19; 30 and 10 us for a 64-pair transfer, which has no constants.
__global__ __launch_bounds__(256) void stage_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                    int n16, const FrameIn* __restrict__ in,
                                                    FrameDev* __restrict__ frames, int n_frames,
                                                    uint32_t* __restrict__ counters) {
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i < kNumCounters) counters[i] = 0u;
    const int n_copy = (n16 + 255) & ~255;             // frames start a workgroup of their own
    if (i < n16) dst[i] = src[i];
    if (i >= n_copy && i - n_copy < n_frames) {
        const FrameIn f = in[i - n_copy];
        frame_constants(f, frames[i - n_copy]);
    }
}

// A table is read through the constant address space (scalar loads): from
// device memory, or, when its pointer is null, from the launch's own
// arguments, where a lone entry is passed by value as the first parameter.
template <class T>
__device__ __forceinline__ cptr<T> lone_arg() {
    return (cptr<T>)__builtin_amdgcn_kernarg_segment_ptr();
}
template <class T>
__device__ __forceinline__ cptr<T> table_or_arg(const T* tab) {
    return tab ? (cptr<T>)tab : lone_arg<T>();
}
struct BatchView {
    cptr<BatchHeader> hdr;
    cptr<KfDev> kfs;
    cptr<FrameDev> frames;
};
__device__ __forceinline__ BatchView batch_view(const BatchHeader* hdr) {
    if (hdr) {
        const cptr<BatchHeader> h = (cptr<BatchHeader>)hdr;
        return {h, (cptr<KfDev>)h->kfs, (cptr<FrameDev>)h->frames};
    }
    const cptr<LoneBatch> a = lone_arg<LoneBatch>();
    return {&a->one.hdr, &a->one.kf, a->frames};
}

__device__ __forceinline__ int divide(int n, const carg<FastDiv>& d) {
    return (int)(__umulhi((unsigned)n << 8, d.m) >> d.l);
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The wavefront's number among the grid's (four wavefronts per workgroup),
// uniform for the compiler, and the grid's count of wavefronts.
__device__ __forceinline__ int grid_wave() {
    return __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
}
__device__ __forceinline__ int grid_waves() { return (int)gridDim.x * 4; }

// ------------------------------------------------------------- init kernel --

// Surfel Initialization section.  Neighbours of new surfel s: surfels that
// are not new, usable, and own a pixel closer than beta_r to u_s.  New
// id_s = mean of Eq. 3 of each neighbour's plane at r_s; new n_s = mean of
// the sign-aligned neighbour normals, renormalised.  Neighbours are visited
// in index order.
//
// A wavefront never spans two keyframes, so the descriptor comes through
// scalar loads (a thread that looked its keyframe up by itself read it with
// chains of vector loads).  Bound by latency: of a new surfel's neighbours
// the is_new bytes come first, then the states of those that count, all in
// flight together.  64 mixed keyframes, half of 1.67 million surfels new:
// 55 us before, 36 now.
__global__ __launch_bounds__(256) void init_kernel(LoneKf, const BatchHeader* __restrict__ hdr_) {
    const BatchView view = batch_view(hdr_);
    const cptr<BatchHeader> hdr = view.hdr;
    const cptr<KfDev> kfs = view.kfs;
    const int lane = threadIdx.x & (kWaveSize - 1);
    __shared__ int s_new_[256 / kWaveSize][kInitSurfels];
    int* const s_new = s_new_[threadIdx.x >> 6];
    const int run = hdr->init_run;
    for (int wv = grid_wave(); wv < hdr->init_waves; wv += grid_waves()) {
        // (keyframes without new surfels take no wavefront)
        int lo = 0, hi = hdr->n_kf - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (kfs[mid].init_wave <= wv) lo = mid; else hi = mid - 1;
        }
        const carg<KfDev>& K = kfs[lo];
        const int gw = K.gw, gh = K.gh;
        const int S = K.patch;
        // the new ones of the wavefront's run of surfels, in order
        int n_new = 0;
        wave_sync();                                       // the previous run's list is read
#pragma unroll
        for (int h = 0; h < kInitSurfels / kWaveSize; ++h) {
            if (h * kWaveSize >= run) break;               // uniform
            const int k = (wv - K.init_wave) * run + h * kWaveSize + lane;
            const bool fresh = k < gw * gh && K.is_new[min(k, gw * gh - 1)] != 0;
            const unsigned long long ball = __ballot(fresh);
            if (fresh) s_new[n_new + __popcll(ball & ((1ull << lane) - 1ull))] = k;
            n_new += __popcll(ball);
        }
        wave_sync();
        for (int k0 = 0; k0 < n_new; k0 += kWaveSize) {
        if (k0 + lane >= n_new) continue;
        const int i = s_new[k0 + lane];
        const int ty = divide(i, K.div_gw), tx = i - ty * gw;
        const float half = 0.5f * (float)(S - 1);
        const float ux = (float)(S * tx) + half, uy = (float)(S * ty) + half;
        const float rsx = (ux - K.cx) / K.fx, rsy = (uy - K.cy) / K.fy;
        const float br = hdr->beta_r > 0.f ? hdr->beta_r : (float)S;
        const float br2 = br * br;
        // a tile dx columns away has its nearest pixel at |dx| S - half from
        // u_s: none beyond floor((br + half) / S) can be closer than br
        const int reach = (int)fminf(floorf((br + half) / (float)S), (float)(gw + gh));
        float id_sum = 0.f, sx = 0.f, sy = 0.f, sz = 0.f, rx = 0.f, ry = 0.f, rz = 0.f;
        int count = 0;
        // one neighbour tile (row ny, column nxt) in visiting order, with its
        // is_new flag, flags and state
        auto visit = [&](int ny, int nxt, uint8_t nw, uint32_t fl, float idj, float njx, float njy,
                         float njz) {
            if (nw) return;
            if (fl & (F_UNINIT | F_DEGENERATE)) return;
            // nearest pixel of tile j to the new surfel's centre
            const float qx = fminf(fmaxf(ux, (float)(S * nxt)), (float)(S * nxt + S - 1));
            const float qy = fminf(fmaxf(uy, (float)(S * ny)), (float)(S * ny + S - 1));
            const float ddx = qx - ux, ddy = qy - uy;
            if (!(ddx * ddx + ddy * ddy < br2)) return;
            const float jx = (float)(S * nxt) + half, jy = (float)(S * ny) + half;
            const float rjx = (jx - K.cx) / K.fx, rjy = (jy - K.cy) / K.fy;
            const float cj = njx * rjx + njy * rjy + njz;
            if (fabsf(cj) < 1e-6f) return;
            // Eq. 3 of plane j at ray r_s: id_j (n_j . r_s) / (n_j . r_j)
            const float id = idj * (njx * rsx + njy * rsy + njz) / cj;
            if (count == 0) { rx = njx; ry = njy; rz = njz; }
            const float sg = (njx * rx + njy * ry + njz * rz) < 0.f ? -1.f : 1.f;
            id_sum += id;
            sx += sg * njx; sy += sg * njy; sz += sg * njz;
            ++count;
        };
        if (reach == 1) {
            // the 3 x 3 neighbourhood (the default radius): every load issued
            // before the first use (out-of-grid slots read the surfel itself
            // and are skipped)
            int js[9];
            bool in[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const int ny = ty - 1 + k / 3, nxt = tx - 1 + k % 3;
                in[k] = ny >= 0 && ny < gh && nxt >= 0 && nxt < gw && k != 4;
                js[k] = in[k] ? ny * gw + nxt : i;
            }
            uint8_t nw[9];
            uint32_t fl[9];
            float idj[9], njx[9], njy[9], njz[9];
#pragma unroll
            for (int k = 0; k < 9; ++k) nw[k] = k == 4 ? 1 : K.is_new[js[k]];
#pragma unroll
            for (int k = 0; k < 9; ++k) in[k] = in[k] && !nw[k];
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                if (!in[k]) continue;
                fl[k] = K.flags[js[k]];
                idj[k] = K.inv_depth[js[k]];
                njx[k] = K.nx[js[k]];
                njy[k] = K.ny[js[k]];
                njz[k] = K.nz[js[k]];
            }
#pragma unroll
            for (int k = 0; k < 9; ++k)
                if (in[k]) visit(ty - 1 + k / 3, tx - 1 + k % 3, nw[k], fl[k], idj[k], njx[k], njy[k], njz[k]);
        } else {
            // one trip to memory per neighbour: its state at once, beside the
            // next one's is_new byte
            const int x0 = max(tx - reach, 0), x1 = min(tx + reach, gw - 1);
            for (int ny = max(ty - reach, 0); ny <= min(ty + reach, gh - 1); ++ny) {
                const int row = ny * gw;
                uint8_t ahead = K.is_new[row + x0];
                for (int nxt = x0; nxt <= x1; ++nxt) {
                    const uint8_t nw = ahead;
                    ahead = K.is_new[row + min(nxt + 1, x1)];
                    if (nw) continue;                  // (so is the surfel itself)
                    const int j = row + nxt;
                    const uint32_t fl = K.flags[j];
                    const float idj = K.inv_depth[j], njx = K.nx[j], njy = K.ny[j], njz = K.nz[j];
                    __asm__ volatile("" ::"v"(fl), "v"(idj), "v"(njx), "v"(njy), "v"(njz));
                    visit(ny, nxt, nw, fl, idj, njx, njy, njz);
                }
            }
        }
        if (count == 0) {
            K.flags[i] |= F_UNINIT;
            continue;
        }
        const float inv = 1.0f / (float)count;
        const float idn = id_sum * inv;
        sx *= inv; sy *= inv; sz *= inv;
        const float l2 = sx * sx + sy * sy + sz * sz;
        if (!(l2 > 0.f) || !(idn > 0.f) || !isfinite(idn) || !isfinite(l2)) {
            K.flags[i] |= F_UNINIT;
            continue;
        }
        const float il = 1.0f / sqrtf(l2);
        K.inv_depth[i] = idn;
        K.nx[i] = sx * il;
        K.ny[i] = sy * il;
        K.nz[i] = sz * il;
        K.flags[i] &= ~F_UNINIT;
        }
    }
}

// --------------------------------------------------------------- GN kernel --

// Cholesky solve of H d = -b in double (textbook form); false when a pivot
// is <= 1e-12 max diag(H), i.e. H is not safely positive definite.
__device__ __forceinline__ bool solve3_fp64(double h00, double h01, double h02, double h11,
                                            double h12, double h22, double b0, double b1,
                                            double b2, double& d0, double& d1, double& d2) {
    const double maxd = fmax(h00, fmax(h11, h22));
    if (!(maxd > 0.0) || !isfinite(maxd)) return false;
    const double tol = 1e-12 * maxd;
    if (!(h00 > tol) || !isfinite(h00)) return false;
    const double l00 = sqrt(h00);
    const double l10 = h01 / l00, l20 = h02 / l00;
    const double p1 = h11 - l10 * l10;
    if (!(p1 > tol) || !isfinite(p1)) return false;
    const double l11 = sqrt(p1);
    const double l21 = (h12 - l20 * l10) / l11;
    const double p2 = h22 - l20 * l20 - l21 * l21;
    if (!(p2 > tol) || !isfinite(p2)) return false;
    const double l22 = sqrt(p2);
    const double y0 = -b0 / l00;
    const double y1 = (-b1 - l10 * y0) / l11;
    const double y2 = (-b2 - l20 * y0 - l21 * y1) / l22;
    d2 = y2 / l22;
    d1 = (y1 - l21 * d2) / l11;
    d0 = (y0 - l10 * d1 - l20 * d2) / l00;
    return true;
}

// Warp constants of one (anchor block, frame) pair, staged in LDS.  The
// plane-induced homography q = H u~ + (K t) id_u (Eq. 6) is evaluated in
// local coordinates: u = u_b + d, with u_b the centre of the aligned
// 16 x 16-pixel anchor block that holds the surfel and d the pixel's offset
// from it (exact, |d| <= 7.5), and an integer anchor (X0, Y0) near the block
// centre's warp at infinite depth, so that every float quantity formed per
// sample is small:
//   x_p - X0 = (Ex + hx0 dx + hx1 dy + kx id_u) / q_z
//   y_p - Y0 = (Ey + hy0 dx + hy1 dy + ky id_u) / q_z
//   q_z      =  Qz + h6 dx  + h7 dy  + k2 id_u
// with Ex = Q_x - X0 Q_z, Q = H u~_b, hx0 = h0 - X0 h6, kx = k0 - X0 k2, ...
// all formed in double once per work item and rounded once to float.  The
// block depends only on the surfel's position, so every launch plan forms
// the same words for a surfel.
constexpr int kPairWords = 12;
enum : int {
    W_HX0 = 0, W_HX1, W_KX, W_EX, W_HY0, W_HY1, W_KY, W_EY, W_QZ, W_X0, W_Y0, W_HZ1
};
// The pair words of every neighbour frame for the anchor point (qbx, qby),
// one frame per lane (lanes below nf), formed in double and rounded once,
// into the wavefront's LDS words.
__device__ __forceinline__ void stage_pair_words(cptr<FrameDev> frames, int nf, int lane,
                                                 double qbx, double qby, float* pairs) {
    if (lane < nf) {
        const gptr<FrameDev> F = (gptr<FrameDev>)(uint64_t)(frames + lane);
        const gptr<double> hm = F->hm;
        const gptr<double> kt = F->kt;
        const double Qx = fma(hm[0], qbx, fma(hm[1], qby, hm[2]));
        const double Qy = fma(hm[3], qbx, fma(hm[4], qby, hm[5]));
        const double Qz = fma(hm[6], qbx, fma(hm[7], qby, hm[8]));
        double X0 = 0.0, Y0 = 0.0;
        if (Qz > 0.0) {
            X0 = rint(fmin(fmax(Qx / Qz, -20000.0), 20000.0));
            Y0 = rint(fmin(fmax(Qy / Qz, -20000.0), 20000.0));
        }
        float* w = pairs + lane * kPairWords;
        w[W_HX0] = (float)(hm[0] - X0 * hm[6]);
        w[W_HX1] = (float)(hm[1] - X0 * hm[7]);
        w[W_KX] = (float)(kt[0] - X0 * kt[2]);
        w[W_EX] = (float)(Qx - X0 * Qz);
        w[W_HY0] = (float)(hm[3] - Y0 * hm[6]);
        w[W_HY1] = (float)(hm[4] - Y0 * hm[7]);
        w[W_KY] = (float)(kt[1] - Y0 * kt[2]);
        w[W_EY] = (float)(Qy - Y0 * Qz);
        w[W_QZ] = (float)Qz;
        w[W_X0] = __int_as_float((int)X0);
        w[W_Y0] = __int_as_float((int)Y0);
        w[W_HZ1] = (float)hm[7];     // h7 again, beside the words the pixel step reads
    }
}

// The four bilinear taps (x0, y0), (x0+1, y0), (x0, y0+1), (x0+1, y0+1) of
// one image, read with buffer loads; the second row uses the row pitch as
// the scalar offset.  f32: one 8-byte load per row.  f16 / u8: one 8-byte
// load per row from the aligned dword below the pair, and a funnel shift (4-
// and 2-byte loads at the pair's own, unaligned address measured 11 % slower
// for the whole kernel).  The tap corner is (row y0, byte column col of x0).
// Two addressings:
//  - by row (BY_ROW: every row pitch of the batch below kMaxRowStride): a
//    structured buffer whose stride is the row pitch, the row as the index
//    and col as the offset, so no multiply forms the address;
//  - raw: the byte offset row x pitch + col.
// The loads run only for samples whose corner passed the validity test
// (x0 < W - 1, y0 < H - 1), so every tap lies inside the image; but the second
// dword of an f16 or u8 load at the row's end can be the one after the image's
// last.  Raw loads are checked dword by dword against the image's bytes (of its
// last row the width, not the pitch: the memory may end there), structured
// ones only by row: the host takes them where that dword is mapped memory
// (rows_by_index_safe).  Its value is not used.
struct Taps {
    float i00, i01, i10, i11;
};

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t image_rsrc(const void* img, unsigned nbytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(img), (short)0, (int)nbytes, 0x00020000);
}
template <typename T, bool BY_ROW>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t image_rsrc_for(const void* img, unsigned pitch_b, unsigned wm1,
                                                                 unsigned hm1) {
    if constexpr (BY_ROW)
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(img), (short)pitch_b, (int)(hm1 + 1), 0x00020000);
    else return image_rsrc(img, (unsigned)image_end((int)wm1 + 1, (int)hm1 + 1, pitch_b, (int)sizeof(T)));
}
// buffer_load_dwordx2 ... idxen offen: base + index x stride + offset + soffset
__device__ u32x2 struct_buffer_load_b64(__amdgpu_buffer_rsrc_t rsrc, int vindex, int voffset, int soffset,
                                        int aux) __asm("llvm.amdgcn.struct.ptr.buffer.load.v2i32");
// the 8 bytes at byte column col of tap rows y0 and y0 + 1
template <bool BY_ROW>
__device__ __forceinline__ void load_row_pair(__amdgpu_buffer_rsrc_t rs, unsigned row, unsigned col,
                                              unsigned pitch_b, u32x2& a, u32x2& b) {
    if constexpr (BY_ROW) {
        a = struct_buffer_load_b64(rs, (int)row, (int)col, 0, 0);
        b = struct_buffer_load_b64(rs, (int)row, (int)col, (int)pitch_b, 0);
    } else {
        const unsigned o = __umul24(row, pitch_b) + col;
        a = __builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, 0);
        b = __builtin_amdgcn_raw_buffer_load_b64(rs, o, pitch_b, 0);
    }
}
// The loaded words of a sample's two tap rows, and their decoding.
struct TapWords {
    u32x2 a, b;
};
template <typename T, bool BY_ROW>
__device__ __forceinline__ TapWords load_words(__amdgpu_buffer_rsrc_t rs, unsigned row, unsigned col,
                                               unsigned pitch_b) {
    TapWords w;
    if constexpr (std::is_same<T, float>::value) load_row_pair<BY_ROW>(rs, row, col, pitch_b, w.a, w.b);
    else load_row_pair<BY_ROW>(rs, row, col & ~3u, pitch_b, w.a, w.b);
    return w;
}
template <typename T>
__device__ __forceinline__ Taps decode_taps(const TapWords& w, unsigned col) {
    Taps t;
    if constexpr (std::is_same<T, float>::value) {
        t.i00 = __uint_as_float(w.a.x);
        t.i01 = __uint_as_float(w.a.y);
        t.i10 = __uint_as_float(w.b.x);
        t.i11 = __uint_as_float(w.b.y);
    } else {
        // u8: the byte shift of v_alignbyte is its third operand mod 4 (the
        // pitch is a multiple of 4, so col's shift is the address's)
        const unsigned pa = __builtin_amdgcn_alignbyte(w.a.y, w.a.x, col);
        const unsigned pb = __builtin_amdgcn_alignbyte(w.b.y, w.b.x, col);
        t.i00 = (float)(pa & 0xffu);
        t.i01 = (float)((pa >> 8) & 0xffu);
        t.i10 = (float)(pb & 0xffu);
        t.i11 = (float)((pb >> 8) & 0xffu);
    }
    return t;
}

// The two row interpolants of a bilinear sample: for each tap row the
// difference d = I(x0+1) - I(x0) and the value I(x0) + ax d.  f32 and u8
// decode the taps first; f16 works on the packed pair directly with mixed
// precision FMAs (the halves convert exactly to float, so the rounding is
// that of the float form).
struct Lerp {
    float d0, top, d1, bot;
};

// hi - lo of a packed pair of halves, in float
__device__ __forceinline__ float half_pair_diff(unsigned pk) {
    float r;
    asm("v_fma_mix_f32 %0, %1, 1.0, -%1 op_sel:[1,0,0] op_sel_hi:[1,0,1]" : "=v"(r) : "v"(pk));
    return r;
}
// a * b + lo (the low half of pk), in float
__device__ __forceinline__ float half_lo_fma(float a, float b, unsigned pk) {
    float r;
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[0,0,1]" : "=v"(r) : "v"(a), "v"(b), "v"(pk));
    return r;
}

template <typename T>
__device__ __forceinline__ Lerp lerp_words(const TapWords& w, unsigned col, float ax) {
    Lerp l;
    if constexpr (std::is_same<T, _Float16>::value) {
        // the byte funnel shift (v_alignbyte) takes its amount mod 4, so col
        // gives the address's shift (the pitch is a multiple of 4)
        const unsigned a = __builtin_amdgcn_alignbyte(w.a.y, w.a.x, col);  // (I(x0), I(x0+1)) of row y0
        const unsigned b = __builtin_amdgcn_alignbyte(w.b.y, w.b.x, col);  // of row y0 + 1
        l.d0 = half_pair_diff(a);
        l.d1 = half_pair_diff(b);
        l.top = half_lo_fma(ax, l.d0, a);
        l.bot = half_lo_fma(ax, l.d1, b);
    } else {
        const Taps t = decode_taps<T>(w, col);
        l.d0 = t.i01 - t.i00;
        l.d1 = t.i11 - t.i10;
        l.top = fmaf(ax, l.d0, t.i00);
        l.bot = fmaf(ax, l.d1, t.i10);
    }
    return l;
}

// floor(x) converted to int in one instruction (v_cvt_flr_i32_f32).
__device__ __forceinline__ int cvt_floor(float x) {
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// One sample from its homogeneous warp q = (nxq, nyq, qz) in local
// coordinates (see the pair words).  sample_warp: projection and validity on
// the integer corner; sample_load: the tap words of a valid sample;
// sample_use: bilinear value and exact gradient, residual, Huber IRLS weight
// and chain factor, accumulating A, B, the valid count and (LAST) the Huber
// cost.
struct Sample {
    float fx, fy, rq;           // x_p - X0, y_p - Y0, 1 / q_z
    unsigned row, col;          // tap corner: row y0, byte column of x0
    bool v;
};
template <typename T>
__device__ __forceinline__ Sample sample_warp(float nxq, float nyq, float qz, const float4& c2, bool pix_ok,
                                              unsigned wm1, unsigned hm1) {
    Sample s;
    s.rq = rcp_fast(qz);
    s.fx = nxq * s.rq;                                    // x_p - X0
    s.fy = nyq * s.rq;                                    // y_p - Y0
    const int flx = cvt_floor(s.fx), fly = cvt_floor(s.fy);
    // unsigned wrap-around: out-of-range (or saturated) corners fail the test
    const unsigned ix = __float_as_uint(c2.y) + (unsigned)flx;
    const unsigned iy = __float_as_uint(c2.z) + (unsigned)fly;
    s.v = pix_ok & (qz > 0.f) & (ix < wm1) & (iy < hm1);
    s.row = iy;
    s.col = ix * (unsigned)sizeof(T);
    return s;
}
template <typename T, bool LAST>
__device__ __forceinline__ void sample_use(const Sample& s, const TapWords& tw, const float4& c0, const float4& c1,
                                           float k2, float ikf, float hk, float img_scale, float& A, float& B,
                                           float& cst, unsigned& nvl, unsigned one) {
    constexpr bool SCALED = std::is_same<T, uint8_t>::value;
    const float ax = __builtin_amdgcn_fractf(s.fx);
    const float ay = __builtin_amdgcn_fractf(s.fy);
    const Lerp l = lerp_words<T>(tw, s.col, ax);
    // bilinear value and the exact gradient of the interpolant
    const float gy = l.bot - l.top;
    const float val = fmaf(ay, gy, l.top);
    const float gx = fmaf(ay, l.d1 - l.d0, l.d0);
    // residual (Eq. 5) and Huber IRLS weight w = min(1, k/|r|) (Eq. 8)
    const float r = SCALED ? fmaf(val, img_scale, -ikf) : val - ikf;
    const float ar = fabsf(r);
    // (the clamp to [0, 1] folds into the multiply; it maps a NaN weight
    // to 0 where min(1, NaN) gives 1, which changes nothing the update
    // reports: B = sum w a r is NaN either way)
    const float wt = fminf(fmaxf(hk * rcp_fast(ar), 0.f), 1.f);
    // dr/did_u = grad I . dpi/dq . K t  (Eq. 8 with dq/did_u = K t):
    // (k0 - x_p k2) = kx - (x_p - X0) k2, likewise for y
    const float tx_ = fmaf(-s.fx, k2, c0.z);
    const float ty_ = fmaf(-s.fy, k2, c1.z);
    const float a = fmaf(gx, tx_, gy * ty_) * (SCALED ? s.rq * img_scale : s.rq);
    const float wa = wt * a;
    A = fmaf(wa, a, A);
    B = fmaf(wa, r, B);
    nvl += one;
    if constexpr (LAST) cst += (ar <= hk) ? 0.5f * r * r : hk * (ar - 0.5f * hk);
}

// The frame loop for the NP pixels of one lane at once: for each neighbour
// frame the frame's constants are read once, the first pixel's warp is
// formed from its offset (dx, dy) from the anchor block centre and its
// inverse depth idu0, and the others' incrementally: pixel j lies dyr rows
// below pixel j-1 of the same surfel and its id_u is didu larger (id_u is
// affine along the column), so its q adds the frame's step, dyr times the
// homography's y column plus didu times K t.  Accumulates A, B and the cost
// per pixel: A = sum w a^2 and B = sum w a r (the per-pixel Jacobian g is
// applied after the loop, hoisted as the paper suggests); the valid counts of the pixels are packed
// one per byte of nvp (pixel j in byte j; at most 16 frames each).
//
// DEEP = 0: each pixel's taps are loaded and used before the next pixel's
// warp, which takes the fewest registers: with seven wavefronts per SIMD the
// others' arithmetic covers each wait.  DEEP = D > 0: the taps of all the
// lane's pixels in D frames are loaded before the first is used, for grids
// that leave a SIMD a wavefront or two and each wait uncovered.  The samples
// and the order of every sum are the same.
//
// SPLIT > 1: a column's pixels are dealt to SPLIT lanes, this lane taking
// rows row0, row0 + SPLIT, ...; (dx, dy) and idu0 are the column's first
// pixel's, and the lane walks the same chain of steps to its own rows.
template <typename T, bool LAST, int NP, bool BY_ROW, int DEEP, int SPLIT>
__device__ __forceinline__ void frame_loop_px(const float* __restrict__ pc, cptr<FrameDev> fr, int nf,
                                              float dx, float dy, float dyr, float idu0, float didu, int row0,
                                              const bool (&pix_ok)[NP],
                                              unsigned pitch_b, unsigned wm1,
                                              unsigned hm1, const float (&ikf)[NP], float hk, float img_scale,
                                              float (&A)[NP], float (&B)[NP], float (&cst)[NP],
                                              unsigned& nvp) {
    static_assert(NP <= 4, "four byte counters");
    constexpr int D = DEEP > 0 ? DEEP : 1;
    for (int f0 = 0; f0 < nf; f0 += D) {
        Sample sm[D][NP];
        TapWords tw[D][NP];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int f = f0 + d;
            if (D > 1 && f >= nf) break;               // wave-uniform
            const float4 c0 = *(const float4*)(pc + f * kPairWords);
            const float4 c1 = *(const float4*)(pc + f * kPairWords + 4);
            const float4 c2 = *(const float4*)(pc + f * kPairWords + 8);
            const float h6 = fr[f].zrow[0], h7 = fr[f].zrow[1], k2 = fr[f].zrow[2];
            const __amdgpu_buffer_rsrc_t rs = image_rsrc_for<T, BY_ROW>(fr[f].img, pitch_b, wm1, hm1);
            // Eq. 6 in local coordinates
            float nxq = fmaf(c0.x, dx, fmaf(c0.y, dy, fmaf(c0.z, idu0, c0.w)));
            float nyq = fmaf(c1.x, dx, fmaf(c1.y, dy, fmaf(c1.z, idu0, c1.w)));
            float qz = fmaf(h6, dx, fmaf(h7, dy, fmaf(k2, idu0, c2.x)));
            // the step to the column's next pixel (formed where it is first
            // used: registers)
            float sx = 0.f, sy = 0.f, sz = 0.f;
            auto step = [&]() {
                sx = fmaf(c0.z, didu, c0.y * dyr);
                sy = fmaf(c1.z, didu, c1.y * dyr);
                sz = fmaf(k2, didu, c2.w * dyr);     // c2.w = h7
            };
            if constexpr (SPLIT > 1) {
                step();
#pragma unroll
                for (int m = 1; m < SPLIT; ++m) {
                    nxq += row0 >= m ? sx : 0.f;
                    nyq += row0 >= m ? sy : 0.f;
                    qz += row0 >= m ? sz : 0.f;
                }
            }
#pragma unroll
            for (int j = 0; j < NP; ++j) {
                if (SPLIT == 1 && j == 1) step();
#pragma unroll
                for (int m = 0; m < (j > 0 ? SPLIT : 0); ++m) {
                    nxq += sx;
                    nyq += sy;
                    qz += sz;
                }
                Sample& s = sm[d][j];
                s = sample_warp<T>(nxq, nyq, qz, c2, pix_ok[j], wm1, hm1);
                if (s.v) {
                    tw[d][j] = load_words<T, BY_ROW>(rs, s.row, s.col, pitch_b);
                    if constexpr (DEEP == 0)
                        sample_use<T, LAST>(s, tw[d][j], c0, c1, k2, ikf[j], hk, img_scale, A[j], B[j], cst[j], nvp,
                                            1u << (8 * j));
                }
            }
        }
        if constexpr (DEEP > 0) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                const int f = f0 + d;
                if (D > 1 && f >= nf) break;
                const float4 c0 = *(const float4*)(pc + f * kPairWords);
                const float4 c1 = *(const float4*)(pc + f * kPairWords + 4);
                const float k2 = fr[f].zrow[2];
#pragma unroll
                for (int j = 0; j < NP; ++j)
                    if (sm[d][j].v)
                        sample_use<T, LAST>(sm[d][j], tw[d][j], c0, c1, k2, ikf[j], hk, img_scale, A[j], B[j], cst[j],
                                            nvp, 1u << (8 * j));
            }
        }
    }
}

// Huber cost (Eq. 5) and valid-sample count of one pixel at a candidate
// state, over all neighbour frames (no Jacobian): the Levenberg-Marquardt
// acceptance test.
// (DEEP as in frame_loop_px: the taps of that many frames in flight.)
template <typename T, bool BY_ROW, int DEEP>
__device__ __forceinline__ void frame_cost(const float* __restrict__ pc, cptr<FrameDev> fr, int nf,
                                           float dx, float dy, float idu, bool pix_ok,
                                           unsigned pitch_b, unsigned wm1,
                                           unsigned hm1, float ikf, float hk, float img_scale,
                                           float& cst, int& nvl) {
    constexpr bool SCALED = std::is_same<T, uint8_t>::value;
    constexpr int D = DEEP > 0 ? DEEP : 1;
    auto use = [&](const Sample& s, const TapWords& w) {
        const Lerp l = lerp_words<T>(w, s.col, __builtin_amdgcn_fractf(s.fx));
        const float val = fmaf(__builtin_amdgcn_fractf(s.fy), l.bot - l.top, l.top);
        const float r = SCALED ? fmaf(val, img_scale, -ikf) : val - ikf;
        const float ar = fabsf(r);
        cst += (ar <= hk) ? 0.5f * r * r : hk * (ar - 0.5f * hk);
        ++nvl;
    };
    for (int f0 = 0; f0 < nf; f0 += D) {
        Sample sm[D];
        TapWords tw[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int f = f0 + d;
            if (D > 1 && f >= nf) break;               // wave-uniform
            const float4 c0 = *(const float4*)(pc + f * kPairWords);
            const float4 c1 = *(const float4*)(pc + f * kPairWords + 4);
            const float4 c2 = *(const float4*)(pc + f * kPairWords + 8);
            const float h6 = fr[f].zrow[0], h7 = fr[f].zrow[1], k2 = fr[f].zrow[2];
            const __amdgpu_buffer_rsrc_t rs = image_rsrc_for<T, BY_ROW>(fr[f].img, pitch_b, wm1, hm1);
            const float nxq = fmaf(c0.x, dx, fmaf(c0.y, dy, fmaf(c0.z, idu, c0.w)));
            const float nyq = fmaf(c1.x, dx, fmaf(c1.y, dy, fmaf(c1.z, idu, c1.w)));
            const float qz = fmaf(h6, dx, fmaf(h7, dy, fmaf(k2, idu, c2.x)));
            sm[d] = sample_warp<T>(nxq, nyq, qz, c2, pix_ok, wm1, hm1);
            if (sm[d].v) {
                tw[d] = load_words<T, BY_ROW>(rs, sm[d].row, sm[d].col, pitch_b);
                if constexpr (DEEP == 0) use(sm[d], tw[d]);
            }
        }
        if constexpr (DEEP > 0) {
#pragma unroll
            for (int d = 0; d < D; ++d)
                if (f0 + d < nf && sm[d].v) use(sm[d], tw[d]);
        }
    }
}

// Per-surfel records exchanged through LDS between the pixel lanes and the
// surfel's owner lane (see gn_kernel).
enum : int {
    // state broadcast to the pixel lanes
    ST_ID = 0, ST_NX, ST_NY, ST_NZ, ST_B1X, ST_B1Y, ST_B1Z, ST_B2X, ST_B2Y, ST_B2Z, ST_INVC,
    ST_RSX, ST_RSY, ST_ALIVE,
    // the owner's own bookkeeping, parked here through the group loop
    ST_FLAGS, ST_LAM, ST_COSTO, ST_NVO, ST_WORDS = 20
};
enum : int {
    // reduced normal equations sent to the owner
    SM_H00 = 0, SM_H01, SM_H02, SM_H11, SM_H12, SM_H22, SM_B0, SM_B1, SM_B2, SM_NV, SM_COST,
    SM_WORDS = 12
};
constexpr int kMaxItemSurfels = 16;

// Tangent basis of n: b1 = normalise(e - (e.n) n), e = x^ if |n_x| < 0.9
// else y^, and b2 = n x b1.
__device__ __forceinline__ void tangent_basis(float nx, float ny, float nz, float& b1x, float& b1y,
                                              float& b1z, float& b2x, float& b2y, float& b2z) {
    const bool ex = fabsf(nx) < 0.9f;
    const float en = ex ? nx : ny;
    b1x = (ex ? 1.f : 0.f) - en * nx;
    b1y = (ex ? 0.f : 1.f) - en * ny;
    b1z = -en * nz;
    const float ib = __frsqrt_rn(b1x * b1x + b1y * b1y + b1z * b1z);
    b1x *= ib; b1y *= ib; b1z *= ib;
    b2x = ny * b1z - nz * b1y;
    b2y = nz * b1x - nx * b1z;
    b2z = nx * b1y - ny * b1x;
}

// One Gauss-Newton step of a surfel on its owner lane, from the reduced
// normal equations sm[] (J^T W J, J^T W r, valid count and cost, laid out as
// SM_*): FEW_SAMPLES below three samples; otherwise the equilibrated 3 x 3
// system (diagonal scaled by 1 + lam) is solved in float by its adjugate, or
// in double by Cholesky when its Frobenius condition exceeds kappa_fp64 or a
// pivot is not safely positive; then id_s += d0 and n = normalise(n + d1 b1 +
// d2 b2) (id_s alone for the depth-only ablation).  Returns true with the
// candidate state when a step is proposed; sets the flags otherwise (a
// rejected step raises lam tenfold when damping is on).
__device__ __forceinline__ bool owner_step(const float* sm, bool alive, bool last,
                                           bool depth_only, bool lm, float kap2, float& lam,
                                           float id, float nx, float ny, float nz, float b1x,
                                           float b1y, float b1z, float b2x, float b2y, float b2z,
                                           uint32_t& flags, float& cost_out, int& nv_out, int& nv,
                                           float& cost_here, float& id_c, float& nx_c,
                                           float& ny_c, float& nz_c) {
    bool cand = false;
    const float H00 = sm[SM_H00], H01 = sm[SM_H01], H02 = sm[SM_H02];
    const float H11 = sm[SM_H11], H12 = sm[SM_H12], H22 = sm[SM_H22];
    const float bb0 = sm[SM_B0], bb1 = sm[SM_B1], bb2 = sm[SM_B2];
    nv = (int)sm[SM_NV];
    cost_here = sm[SM_COST];
    if (alive && last) cost_out = cost_here;
    if (alive) {
        nv_out = nv;
        float d0s = 0.f, d1s = 0.f, d2s = 0.f;
        bool ok = true;
        if (nv < 3) {
            flags |= F_FEW_SAMPLES;
            ok = false;
        }
        const float dd = 1.f + lam;          // (H + lam diag H): equilibrated diagonal
        if (ok && depth_only) {
            if (H00 > 0.f && isfinite(H00)) {
                d0s = -bb0 * rcp_fast(H00 * dd);
            } else {
                flags |= F_SOLVE_FAIL;
                ok = false;
            }
        } else if (ok) {
            // equilibrate: E = D^-1/2 H D^-1/2 (unit diagonal).  The float
            // solve is formed unconditionally (no branches: the tests below
            // are combined with |) and replaced by the double-precision one
            // where a diagonal is not positive and finite or the system is
            // too ill-conditioned for float.
            const float maxd = fmaxf(H00, fmaxf(H11, H22));
            const float e0 = __frsqrt_rn(H00), e1 = __frsqrt_rn(H11), e2 = __frsqrt_rn(H22);
            const float e01 = H01 * e0 * e1, e02 = H02 * e0 * e2, e12 = H12 * e1 * e2;
            // adjugate and determinant of E (diagonal dd = 1 + lambda)
            const float d2 = dd * dd;
            const float c00 = fmaf(-e12, e12, d2), c11 = fmaf(-e02, e02, d2);
            const float c22 = fmaf(-e01, e01, d2);
            const float c01 = fmaf(e02, e12, -dd * e01), c02 = fmaf(e01, e12, -dd * e02);
            const float c12 = fmaf(e01, e02, -dd * e12);
            const float det = fmaf(e01, c01, fmaf(e02, c02, dd * c00));
            // kappa_F(E)^2 = ||E||_F^2 ||adj E||_F^2 / det^2  (>= kappa_2(E)^2)
            const float fro2 = 3.f * d2 + 2.f * (e01 * e01 + e02 * e02 + e12 * e12);
            const float adj2 = c00 * c00 + c11 * c11 + c22 * c22 +
                               2.f * (c01 * c01 + c02 * c02 + c12 * c12);
            // raw Cholesky pivots are H_jj times the equilibrated ones
            const float p1 = c22 * rcp_fast(dd);   // dd - e01^2 / dd (only compared)
            const float p2 = det * rcp_fast(c22);  // (only compared)
            const bool need64 = !(H00 > 0.f) | !(H11 > 0.f) | !(H22 > 0.f) | !isfinite(maxd) |
                                !(fro2 * adj2 <= kap2 * det * det) | !(det > 0.f) | !(c22 > 0.f) |
                                !(H11 * p1 > 1e-10f * maxd * dd) | !(H22 * p2 > 1e-10f * maxd * dd);
            {
                const float bh0 = bb0 * e0, bh1 = bb1 * e1, bh2 = bb2 * e2;
                const float idet = rcp_fast(det);
                d0s = -(c00 * bh0 + c01 * bh1 + c02 * bh2) * idet * e0;
                d1s = -(c01 * bh0 + c11 * bh1 + c12 * bh2) * idet * e1;
                d2s = -(c02 * bh0 + c12 * bh1 + c22 * bh2) * idet * e2;
            }
            if (need64) {
                flags |= F_FP64_SOLVE;
                double dd0 = 0.0, dd1 = 0.0, dd2 = 0.0;
                const double dmp = 1.0 + (double)lam;
                if (solve3_fp64((double)H00 * dmp, H01, H02, (double)H11 * dmp, H12,
                                (double)H22 * dmp, bb0, bb1, bb2, dd0, dd1, dd2)) {
                    d0s = (float)dd0; d1s = (float)dd1; d2s = (float)dd2;
                } else {
                    flags |= F_SOLVE_FAIL;
                    ok = false;
                }
            }
        }
        if (ok) {
            // update: id_s += d0; n = normalise(n + d1 b1 + d2 b2) (the
            // depth-only ablation moves id_s alone and keeps n)
            id_c = id + d0s;
            nx_c = nx; ny_c = ny; nz_c = nz;
            bool ok_step;
            if (depth_only) {
                ok_step = (id_c > 0.f) && isfinite(id_c);
            } else {
                const float mx = fmaf(d1s, b1x, fmaf(d2s, b2x, nx));
                const float my = fmaf(d1s, b1y, fmaf(d2s, b2y, ny));
                const float mz = fmaf(d1s, b1z, fmaf(d2s, b2z, nz));
                const float l2 = mx * mx + my * my + mz * mz;
                ok_step = (id_c > 0.f) && isfinite(id_c) && (l2 > 0.f) && isfinite(l2);
                if (ok_step) {
                    const float il = __frsqrt_rn(l2);
                    nx_c = mx * il; ny_c = my * il; nz_c = mz * il;
                }
            }
            if (!ok_step) {
                flags |= F_REJECTED;
                if (lm) lam *= 10.f;
            } else {
                cand = true;
            }
        }
    }
    return cand;
}

// Levenberg-Marquardt acceptance of a candidate on its owner lane: the
// candidate's cost cost2 over nv2 valid samples against the current cost
// over nv.  Accepted when the mean Huber cost per valid sample does not rise
// (cost2 / nv2 <= cost / nv, compared as cost2 nv <= cost nv2) and at least
// three samples remain.  lam shrinks tenfold (floor 1e-9) on acceptance and
// grows tenfold on refusal.
__device__ __forceinline__ bool lm_accept(float cost2, int nv2, float cost_here, int nv, float& lam) {
    if (nv2 < 3 || !(cost2 * (float)nv <= cost_here * (float)nv2)) {
        lam *= 10.f;
        return false;
    }
    lam = fmaxf(lam * 0.1f, 1e-9f);
    return true;
}

// The candidate's Huber cost and valid count over a column whose NP * SPLIT
// pixels are dealt to SPLIT lanes (see frame_loop_px).  The column's cost is
// one chain of additions, pixel by pixel and frame by frame; each lane forms
// its pixels' terms with the taps of four frames in flight and leaves them in
// LDS (terms: the lane's words, 64 apart; a sample that is not valid is a term
// of zero, which changes no sum), and the lanes then add theirs in turn, the
// running sum handed from row to row.  The column's cost ends in the lane of
// the last row.  A lone damped 333 x 251 keyframe of five neighbours: 166 us
// per call with two frames in flight on unsplit columns, 97 split over four
// lanes.
template <typename T, bool BY_ROW, int NP, int SPLIT>
__device__ __forceinline__ void split_cost(const float* __restrict__ pc, cptr<FrameDev> fr, int nf, float dx,
                                           const float (&dy)[NP], const float (&idu)[NP], const bool (&pix_ok)[NP],
                                           unsigned pitch_b, unsigned wm1, unsigned hm1, const float (&ikf)[NP],
                                           float hk, float img_scale, int row0, float4* terms, float& cst,
                                           int& nvl) {
    constexpr bool SCALED = std::is_same<T, uint8_t>::value;
    constexpr int D = 4, C = kMaxNbr / D;
    for (int f0 = 0; f0 < nf; f0 += D) {
        Sample sm[D][NP];
        TapWords tw[D][NP];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int f = f0 + d;
#pragma unroll
            for (int j = 0; j < NP; ++j) sm[d][j].v = false;
            if (f < nf) {                              // wave-uniform
                const float4 c0 = *(const float4*)(pc + f * kPairWords);
                const float4 c1 = *(const float4*)(pc + f * kPairWords + 4);
                const float4 c2 = *(const float4*)(pc + f * kPairWords + 8);
                const float h6 = fr[f].zrow[0], h7 = fr[f].zrow[1], k2 = fr[f].zrow[2];
                const __amdgpu_buffer_rsrc_t rs = image_rsrc_for<T, BY_ROW>(fr[f].img, pitch_b, wm1, hm1);
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    const float nxq = fmaf(c0.x, dx, fmaf(c0.y, dy[j], fmaf(c0.z, idu[j], c0.w)));
                    const float nyq = fmaf(c1.x, dx, fmaf(c1.y, dy[j], fmaf(c1.z, idu[j], c1.w)));
                    const float qz = fmaf(h6, dx, fmaf(h7, dy[j], fmaf(k2, idu[j], c2.x)));
                    Sample& s = sm[d][j];
                    s = sample_warp<T>(nxq, nyq, qz, c2, pix_ok[j], wm1, hm1);
                    if (s.v) tw[d][j] = load_words<T, BY_ROW>(rs, s.row, s.col, pitch_b);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            float t[D];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                t[d] = 0.f;
                const Sample& s = sm[d][j];
                if (s.v) {
                    const Lerp l = lerp_words<T>(tw[d][j], s.col, __builtin_amdgcn_fractf(s.fx));
                    const float val = fmaf(__builtin_amdgcn_fractf(s.fy), l.bot - l.top, l.top);
                    const float r = SCALED ? fmaf(val, img_scale, -ikf[j]) : val - ikf[j];
                    const float ar = fabsf(r);
                    t[d] = (ar <= hk) ? 0.5f * r * r : hk * (ar - 0.5f * hk);
                    ++nvl;
                }
            }
            terms[(j * C + f0 / D) * kWaveSize] = make_float4(t[0], t[1], t[2], t[3]);
        }
    }
    {
#pragma clang fp contract(off)
#pragma unroll
        for (int m = 0; m < NP * SPLIT; ++m) {
            // lane i takes the running sum of lane i -+ 4, the row before
            if (m > 0) cst = SPLIT == 2 && m % 2 == 0 ? dpp_f<0x104>(cst) : dpp_f<0x114>(cst);
            for (int c = 0; c < (nf + D - 1) / D; ++c) {
                const float4 t = terms[((m / SPLIT) * C + c) * kWaveSize];
                cst += t.x; cst += t.y; cst += t.z; cst += t.w;
            }
        }
    }
}

// The fused Gauss-Newton kernel.
//
// Mapping.  A work item is a block of surfels inside one aligned anchor
// block (16 x 16 pixels): K groups, each filling the 64 lanes of the
// wavefront with pixels (S = 4: a TX x TY arrangement of four, eight or
// sixteen 4 x 4 surfels, 16, 8 or 4 lanes per surfel, one, two or four
// pixels per lane; S = 8: one 8 x 8 surfel; S = 16: one 16 x 16 surfel,
// four pixels per lane).  Per iteration the wavefront walks its groups; for
// each, every lane forms the frame-independent terms of its pixels' surfel
// (hoisted as the paper suggests), loops over the neighbour frames (warp,
// bilinear sample and gradient, Huber-weighted residual, chain factor) and
// the surfel's lanes reduce J^T W J and J^T W r with DPP.  Each surfel has
// an owner lane (lane k among the surfel's lanes for group k); the owners
// then solve all K groups' 3 x 3 systems at once, so the per-surfel work
// (solve, update, tangent basis) is issued once per K groups.  Sums and states pass
// between the pixel lanes and the owners through LDS.  All iterations run in
// the kernel: surfels never read each other during the optimisation.
// Registers are the budget that matters (the kernel issues a VALU
// instruction on nearly every cycle it can, and more wavefronts per SIMD
// hide the rest): values that the frame loop does not use are not held
// through it but formed again or read back from LDS afterwards.  BY_ROW
// reads the neighbour rows by index (row pitches below kMaxRowStride).
//
// Wavefronts per SIMD each plan's kernel is compiled for (the register
// budget: 72 VGPRs for seven, 80 for six, 96 for five).  One sample at a time
// and one group, four pixels per lane, is the form of large damped batches: 64
// mixed u8 keyframes take 8.00 ms at five, 8.07 at six, 7.92 at seven and 8.65
// at eight, where it spills inside the iteration loop; 32 of 16 x 16 surfels
// 2.72, 2.71, 2.65, 2.71.  Undamped, in the plans of fewer pixels per lane, and
// in bounded persistent grids occupancy pays more (f16 4x4 one group 4.69 ms at
// four, 4.30 at five, 3.94 at six, 3.76 at seven, 4.05 at eight).
// The DEEP forms keep more samples in registers: two frames of four pixels
// take 125 VGPRs (four wavefronts), one frame 96 (five), the SPLIT forms 92
// and, damped, up to 129 (the two-lane form's terms leave LDS for three
// wavefronts anyway).
template <int S, int K, int DEEP, int SPLIT>
constexpr int gn_waves() {
    return SPLIT > 1 ? 4 : DEEP == 2 ? 2 : DEEP == 1 ? 5 : K == 1 ? 7 : (S == 8 ? 6 : 5);
}

template <typename T, int S, int TX, int TY, int K, bool BY_ROW, int DEEP, int SPLIT, bool PERSIST, bool DAMPED>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(gn_waves<S, K, DEEP, SPLIT>(), 8))) void gn_kernel(LoneBatch,
                                                           const BatchHeader* __restrict__ hdr_,
                                                           uint32_t* __restrict__ counters) {
    constexpr ItemGeo G = item_geo(S, TX, TY, K);
    constexpr int PIX = S * S;                                // pixels per surfel
    constexpr int SLOTS = TX * TY;                            // surfels per group
    constexpr int LANES = kWaveSize / SLOTS;                  // lanes per surfel
    constexpr int PPL = PIX / LANES;                          // pixels per lane
    constexpr int NS = K * SLOTS;                             // surfels per work item
    constexpr int RL = LANES / SPLIT;                         // lanes that join in a surfel's sums
    // rows from one pixel of a column's chain to the next
    constexpr float DYR = SPLIT > 1 ? 1.f : (float)(LANES / S);
    static_assert(SPLIT == 1 || (S == 4 && K == 1 && PPL * SPLIT == 4 && LANES == S * SPLIT), "split columns");
    static_assert(PPL * LANES == PIX, "a group fills the wavefront");
    static_assert(PPL == 1 || LANES % S == 0, "a lane's pixels share a column");
    static_assert(NS <= kMaxItemSurfels && K <= LANES, "surfels per item");
    static_assert(G.ix <= G.ab && G.iy <= G.ab, "a work item lies in one anchor block");
    const BatchView view = batch_view(hdr_);
    const cptr<BatchHeader> hdr = view.hdr;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    // pixel role: slot r of a group; pixels p + LANES j (j < PPL) of that surfel
    const int r = lane / LANES;
    const int p = lane % LANES;
    const float half = 0.5f * (float)(S - 1);
    const int row0 = SPLIT > 1 ? p / S : 0;      // the lane's first row in its column's chain
    int pxs[PPL], pys[PPL];
    float dxp[PPL], dyp[PPL];                    // offsets from u_s (exact)
#pragma unroll
    for (int j = 0; j < PPL; ++j) {
        const int q = p + LANES * j;
        pxs[j] = q % S;
        pys[j] = q / S;
        dxp[j] = (float)pxs[j] - half;
        dyp[j] = (float)pys[j] - half;
    }
    // owner role: surfel (group ok_g, slot ok_r) of the item
    const int ok_g = SLOTS == 1 ? lane : lane & (LANES - 1);
    const int ok_r = SLOTS == 1 ? 0 : lane >> __builtin_ctz(LANES);
    const bool owner = ok_g < K;
    const int own = ok_g * SLOTS + ok_r;

    const int n_kf = hdr->n_kf;
    const int total = hdr->total_items;
    const int iters = hdr->iters;
    const float hk = hdr->huber_k;
    const float kappa_s = hdr->kappa_fp64;
    const bool depth_only = hdr->depth_only != 0;
    const uint32_t stamp = hdr->stamp;
    const float lm0 = hdr->lm_lambda;
    const bool lm = DAMPED && lm0 > 0.f;
    const cptr<KfDev> kfs = view.kfs;

    __shared__ float4 s_pairs[kBlockThreads / kWaveSize][kMaxNbr * kPairWords / 4];
    __shared__ float4 s_state[kBlockThreads / kWaveSize][kMaxItemSurfels * ST_WORDS / 4];
    __shared__ float4 s_sums[kBlockThreads / kWaveSize][kMaxItemSurfels * SM_WORDS / 4];
    float* const pairs = (float*)s_pairs[wave];
    float* const lst = (float*)s_state[wave];
    float* const lsm = (float*)s_sums[wave];
    // a split column's candidate costs, frame by frame (split_cost)
    constexpr int TERMS = DAMPED && SPLIT > 1 ? PPL * kMaxNbr / 4 * kWaveSize : 1;
    __shared__ float4 s_terms[kBlockThreads / kWaveSize][TERMS];

    int q = PERSIST ? (int)(blockIdx.x % (unsigned)kXcds) % hdr->n_queues : 0;
    int q_left = hdr->n_queues;
    int hint = 0;
    int item;
    if constexpr (PERSIST) {
        item = pull_item(hdr, counters, q, q_left, lane, total);
    } else if (hdr->n_queues == kXcds) {
        // one share of the work items per XCD: the hardware hands the
        // workgroups to the XCDs in turn, so workgroup b runs on XCD
        // b % kXcds and takes that share's items in order (every item is
        // still taken once under any other dispatch order; only the L2
        // locality depends on it)
        const int share = (int)(blockIdx.x % (unsigned)kXcds);
        const int it = hdr->queues[share].begin +
                       (int)(blockIdx.x / (unsigned)kXcds) * (kBlockThreads / kWaveSize) + wave;
        item = it < hdr->queues[share].end ? it : total;
    } else {
        item = blockIdx.x * (kBlockThreads / kWaveSize) + wave;
    }
    for (; item < total; item = PERSIST ? pull_item(hdr, counters, q, q_left, lane, total) : total) {
        item = __builtin_amdgcn_readfirstlane(item);
        const int kidx = find_kf(kfs, n_kf, item, hint);
        hint = kidx;
        const cptr<KfDev> Kd = kfs + kidx;
        // item -> anchor block (bx, by) and the item's place in it
        const int g = item - Kd->item_base;
        const int blk = g / G.ipb, sub = g - blk * G.ipb;
        const int bx = blk % Kd->groups_x, by = blk / Kd->groups_x;
        const int it0x = bx * G.ab + (sub % (G.ab / G.ix)) * G.ix;
        const int it0y = by * G.ab + (sub / (G.ab / G.ix)) * G.iy;
        const int gw = Kd->gw, gh = Kd->gh;
        if (it0x >= gw || it0y >= gh) continue;          // item entirely outside the grid
        const int nf = Kd->n_nbr;
        const float img_scale = Kd->img_scale;
        const unsigned pitch_b = (unsigned)Kd->nbr_pitch_b;
        const unsigned wm1 = (unsigned)(Kd->width - 1), hm1 = (unsigned)(Kd->height - 1);
        const float fxk = Kd->fx, fyk = Kd->fy, cxk = Kd->cx, cyk = Kd->cy;
        // r_u - r_s of the lane's first pixel; its later pixels lie DYR rows
        // apart in the same column, dyr_f apart in r
        const float drx0 = dxp[0] / fxk, dry0 = (SPLIT > 1 ? -half : dyp[0]) / fyk;
        const float dyr_f = DYR / fyk;
        // anchor block centre (pixels)
        const int bpx = bx * G.ab * S, bpy = by * G.ab * S;
        {
            // warp constants of every frame for this anchor block, one frame
            // per lane, in double
            wave_sync();
            stage_pair_words(view.frames + Kd->frame_base, nf, lane,
                             (double)bpx + 0.5 * (double)(G.ab * S - 1),
                             (double)bpy + 0.5 * (double)(G.ab * S - 1), pairs);
        }
        // the frame table pointer is wave-uniform: keep it in SGPRs
        const uint64_t fr_bits = (uint64_t)(view.frames + Kd->frame_base);
        const uint32_t fr_lo = __builtin_amdgcn_readfirstlane((uint32_t)fr_bits);
        const uint32_t fr_hi = __builtin_amdgcn_readfirstlane((uint32_t)(fr_bits >> 32));
        const cptr<FrameDev> fr = (cptr<FrameDev>)(((uint64_t)fr_hi << 32) | fr_lo);

        // pixel lanes: keyframe value of this lane's pixels in every group
        float ikf[K][PPL];
        const gptr<T> kimg = (gptr<T>)Kd->kf_img;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int tx = it0x + (k % G.gx) * TX + r % TX, ty = it0y + (k / G.gx) * TY + r / TX;
#pragma unroll
            for (int j = 0; j < PPL; ++j) {
                ikf[k][j] = 0.f;
                if (tx < gw && ty < gh)
                    ikf[k][j] = ldg<T>(kimg + ((unsigned)(S * ty + pys[j]) * (unsigned)Kd->kf_pitch +
                                               (unsigned)(S * tx + pxs[j]))) * Kd->kf_scale;
            }
        }

        // owner lanes: the surfel's state
        const int otx = it0x + (ok_g % G.gx) * TX + ok_r % TX;
        const int oty = it0y + (ok_g / G.gx) * TY + ok_r / TX;
        const bool own_ok = owner && otx < gw && oty < gh;
        const int sidx = oty * gw + otx;
        const float usx = (float)(S * otx) + half, usy = (float)(S * oty) + half;
        const float rsx = (usx - cxk) / fxk, rsy = (usy - cyk) / fyk;   // r_s (z = 1)
        float id = 0.f, nx = 0.f, ny = 0.f, nz = -1.f;
        uint32_t flags = 0u;
        if (own_ok) {
            id = ((gptr<float>)Kd->inv_depth)[sidx];
            nx = ((gptr<float>)Kd->nx)[sidx];
            ny = ((gptr<float>)Kd->ny)[sidx];
            nz = ((gptr<float>)Kd->nz)[sidx];
            flags = ((gptr<uint32_t>)Kd->flags)[sidx] & ~F_GN_BITS;
        }
        bool alive = own_ok;
        bool updated = false;
        float cost_out = 0.f;
        int nv_out = 0;
        float lam = lm0;             // Levenberg-Marquardt damping of this surfel
        float b1x = 0.f, b1y = 0.f, b1z = 0.f, b2x = 0.f, b2y = 0.f, b2z = 0.f;
        // r_s is the item's: written once (the words are the previous item's
        // until the sync before the pair words, which is behind us)
        if (owner) {
            float* o = lst + own * ST_WORDS;
            o[ST_RSX] = rsx; o[ST_RSY] = rsy;
        }

        for (int it = 0; it < iters; ++it) {
            const bool last = (it == iters - 1);
            // the cost is summed on the last iteration and for the damped
            // variant: a wave-uniform flag, kept in a scalar register
            const bool with_cost = __builtin_amdgcn_readfirstlane((int)(last || lm)) != 0;
            // ---- owners: degeneracy, tangent basis, broadcast of the state
            if (owner) {
                const float* os = lst + own * ST_WORDS;
                const float c = nx * os[ST_RSX] + ny * os[ST_RSY] + nz;     // n . r_s
                if (alive && fabsf(c) < 1e-6f) {
                    flags |= F_DEGENERATE;
                    alive = false;
                    cost_out = 0.f;
                    nv_out = 0;
                }
                tangent_basis(nx, ny, nz, b1x, b1y, b1z, b2x, b2y, b2z);
                float* o = lst + own * ST_WORDS;
                o[ST_ID] = id; o[ST_NX] = nx; o[ST_NY] = ny; o[ST_NZ] = nz;
                o[ST_B1X] = b1x; o[ST_B1Y] = b1y; o[ST_B1Z] = b1z;
                o[ST_B2X] = b2x; o[ST_B2Y] = b2y; o[ST_B2Z] = b2z;
                o[ST_INVC] = rcp_fast(c);                    // |c| >= 1e-6 where used
                o[ST_ALIVE] = alive ? 1.f : 0.f;
                o[ST_FLAGS] = __uint_as_float(flags); o[ST_LAM] = lam;
                o[ST_COSTO] = cost_out; o[ST_NVO] = __int_as_float(nv_out);
            }
            wave_sync();
            // ---- pixel lanes: linearise every group and reduce per surfel
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const float* st = lst + (k * SLOTS + r) * ST_WORDS;
                const float4 sa = *(const float4*)(st + 0);      // id, nx, ny, nz
                const float sid = sa.x, snx = sa.y, sny = sa.z;
                const float inv_c = st[ST_INVC];
                const bool salive = st[ST_ALIVE] != 0.f;
                const int tx = it0x + (k % G.gx) * TX + r % TX, ty = it0y + (k / G.gx) * TY + r / TX;
                // this lane's share of J^T W J = sum_u A_u g g^T and
                // J^T W r = sum_u B_u g (the frame sum hoisted), its valid
                // count and cost, over its pixels in order
                float ph[9], pnv, pcs;
                // frame-independent per-pixel terms (Eq. 3, Eq. 9)
                bool pix_ok[PPL];
                // sigma_u = n . (r_u - r_s) / (n . r_s): the lane's first
                // pixel's, and the step between its pixels (same column);
                // id_u = id_s (1 + sigma_u) steps by id_s dsig
                const float cnx = snx * inv_c, cny = sny * inv_c;
                const float sig0 = fmaf(cny, dry0, cnx * drx0);
                const float dsig = cny * dyr_f;
                const float idu0 = fmaf(sid, sig0, sid);
                const float didu = sid * dsig;
#pragma unroll
                for (int j = 0; j < PPL; ++j) {
                    const int row = row0 + SPLIT * j;
                    const float sig = row == 0 ? sig0 : fmaf((float)row, dsig, sig0);
                    pix_ok[j] = salive && (fmaf(sid, sig, sid) > 0.f);
                }
                // the first pixel's offset from the anchor block centre; the
                // lane's later pixels lie DYR rows apart in the same column
                const float bdx = (float)(S * tx + pxs[0] - bpx) - 0.5f * (float)(G.ab * S - 1);
                const float bdy = (float)(S * ty + (SPLIT > 1 ? 0 : pys[0]) - bpy) - 0.5f * (float)(G.ab * S - 1);
                float Ap[PPL], Bp[PPL], cp[PPL];
                unsigned nvp = 0u;
#pragma unroll
                for (int j = 0; j < PPL; ++j) {
                    Ap[j] = 0.f; Bp[j] = 0.f; cp[j] = 0.f;
                }
                if (with_cost)
                    frame_loop_px<T, true, PPL, BY_ROW, DEEP, SPLIT>(pairs, fr, nf, bdx, bdy, DYR, idu0, didu, row0, pix_ok, pitch_b,
                                                wm1, hm1, ikf[k], hk, img_scale, Ap, Bp, cp, nvp);
                else
                    frame_loop_px<T, false, PPL, BY_ROW, DEEP, SPLIT>(pairs, fr, nf, bdx, bdy, DYR, idu0, didu, row0, pix_ok, pitch_b,
                                                 wm1, hm1, ikf[k], hk, img_scale, Ap, Bp, cp, nvp);
                // the surfel's state and tangent basis, read again from LDS
                // after the frame loop rather than held in registers through it
                __asm__ volatile("" ::: "memory");
                const float4 sa2 = *(const float4*)(st + 0);     // id, nx, ny, nz
                const float4 sb = *(const float4*)(st + 4);      // b1, b2x
                const float4 sc = *(const float4*)(st + 8);      // b2y, b2z, 1/c, rsx
                const float srsy = st[ST_RSY];
                const float sb1x = sb.x, sb1y = sb.y, sb1z = sb.z;
                const float sb2x = sb.w, sb2y = sc.x, sb2z = sc.y, srsx = sc.w;
                const float pinv_c = sc.z;
                // g_u = (1 + sigma_u, kk b1 . d_u, kk b2 . d_u) with
                // d_u = (r_u - r_s) - sigma_u (r_s, 1) and kk = id_s / (n . r_s):
                // b . d_u = (b_x drx + b_y dry_u) - sigma_u (b . (r_s, 1)).  All
                // three are affine in the pixel's row, so each is its value at
                // the lane's first pixel plus j steps.  The depth-only ablation
                // zeroes kk, and with it the normal columns.
                const float pcnx = sa2.y * pinv_c, pcny = sa2.z * pinv_c;
                const float psig0 = fmaf(pcny, dry0, pcnx * drx0);
                const float pdsig = pcny * dyr_f;
                const float kk = depth_only ? 0.f : sa2.x * pinv_c;
                const float k1x = kk * sb1x, k1y = kk * sb1y, k2x = kk * sb2x, k2y = kk * sb2y;
                const float q1 = kk * fmaf(sb1x, srsx, fmaf(sb1y, srsy, sb1z));
                const float q2 = kk * fmaf(sb2x, srsx, fmaf(sb2y, srsy, sb2z));
                const float g00 = 1.f + psig0;
                const float g10 = fmaf(-psig0, q1, fmaf(k1y, dry0, k1x * drx0));
                const float g20 = fmaf(-psig0, q2, fmaf(k2y, dry0, k2x * drx0));
                const float dg1 = fmaf(-pdsig, q1, k1y * dyr_f);
                const float dg2 = fmaf(-pdsig, q2, k2y * dyr_f);
                // the lane's valid samples: the byte counters summed (v_sad_u8)
                unsigned nvs = __builtin_amdgcn_sad_u8(nvp, 0u, 0u);
                // the column's sums, brought to the lane of its first row
                constexpr int NC = PPL * SPLIT;
                float A[NC], B[NC], cst[NC];
#pragma unroll
                for (int j = 0; j < PPL; ++j) {
                    A[SPLIT * j] = Ap[j]; B[SPLIT * j] = Bp[j]; cst[SPLIT * j] = cp[j];
                    if constexpr (SPLIT >= 2) {
                        A[SPLIT * j + 1] = dpp_f<0x104>(Ap[j]);      // row_shl:4 (lane i takes lane i + 4)
                        B[SPLIT * j + 1] = dpp_f<0x104>(Bp[j]);
                        cst[SPLIT * j + 1] = dpp_f<0x104>(cp[j]);
                    }
                    if constexpr (SPLIT == 4) {
                        A[2] = dpp_f<0x108>(Ap[j]); A[3] = dpp_f<0x10C>(Ap[j]);
                        B[2] = dpp_f<0x108>(Bp[j]); B[3] = dpp_f<0x10C>(Bp[j]);
                        cst[2] = dpp_f<0x108>(cp[j]); cst[3] = dpp_f<0x10C>(cp[j]);
                    }
                }
                if constexpr (SPLIT == 2) nvs += (unsigned)dpp_i<0x104>((int)nvs);
                if constexpr (SPLIT == 4)
                    nvs += (unsigned)(dpp_i<0x104>((int)nvs) + dpp_i<0x108>((int)nvs) + dpp_i<0x10C>((int)nvs));
                if constexpr (NC == 4) {
                    // sum_j A_j g_j g_j^T and sum_j B_j g_j with g_j = ga + j gb,
                    // through the lane's moments S_m = sum_j j^m A_j and
                    // T_m = sum_j j^m B_j: with u = S0 ga + S1 gb and
                    // v = S1 ga + S2 gb, H = u ga^T + v gb^T and b = T0 ga + T1 gb
                    // (42 instructions for the four pixels against 60 per pixel)
                    const float S0 = (A[0] + A[1]) + (A[2] + A[3]);
                    const float S1 = fmaf(3.f, A[3], fmaf(2.f, A[2], A[1]));
                    const float S2 = fmaf(9.f, A[3], fmaf(4.f, A[2], A[1]));
                    const float T0 = (B[0] + B[1]) + (B[2] + B[3]);
                    const float T1 = fmaf(3.f, B[3], fmaf(2.f, B[2], B[1]));
                    const float ga[3] = {g00, g10, g20}, gb[3] = {pdsig, dg1, dg2};
                    float uu[3], vv[3];
#pragma unroll
                    for (int a = 0; a < 3; ++a) {
                        uu[a] = fmaf(S1, gb[a], S0 * ga[a]);
                        vv[a] = fmaf(S2, gb[a], S1 * ga[a]);
                    }
                    ph[0] = fmaf(vv[0], gb[0], uu[0] * ga[0]);     // H00
                    ph[1] = fmaf(vv[0], gb[1], uu[0] * ga[1]);     // H01
                    ph[2] = fmaf(vv[0], gb[2], uu[0] * ga[2]);     // H02
                    ph[3] = fmaf(vv[1], gb[1], uu[1] * ga[1]);     // H11
                    ph[4] = fmaf(vv[1], gb[2], uu[1] * ga[2]);     // H12
                    ph[5] = fmaf(vv[2], gb[2], uu[2] * ga[2]);     // H22
#pragma unroll
                    for (int a = 0; a < 3; ++a) ph[6 + a] = fmaf(T1, gb[a], T0 * ga[a]);
                    pcs = (cst[0] + cst[1]) + (cst[2] + cst[3]);
                } else {
#pragma unroll
                    for (int j = 0; j < PPL; ++j) {
                        const float g0 = fmaf((float)j, pdsig, g00);
                        const float g1 = fmaf((float)j, dg1, g10);
                        const float g2 = fmaf((float)j, dg2, g20);
                        const float ag0 = A[j] * g0, ag1 = A[j] * g1, ag2 = A[j] * g2;
                        const float u[9] = {ag0, ag0, ag0, ag1, ag1, ag2, B[j], B[j], B[j]};
                        const float v[9] = {g0, g1, g2, g1, g2, g2, g0, g1, g2};
#pragma unroll
                        for (int e = 0; e < 9; ++e) ph[e] = (j == 0) ? u[e] * v[e] : fmaf(u[e], v[e], ph[e]);
                        pcs = (j == 0) ? cst[j] : pcs + cst[j];
                    }
                }
                pnv = (float)nvs;
                // reduced two at a time: lane 0 of the surfel ends with words
                // 0, 2, 4, 6, 8 and lane 1 with words 1, 3, 5, 7, 9 (the valid
                // count as an exact float)
                float s0, s1, s2, s3, s4;
                {
                    // No FMA contraction: each butterfly step must be a plain
                    // add of two rounded values so that the sums do not depend
                    // on which lane forms them.
#pragma clang fp contract(off)
                    const bool odd = (p & 1) != 0;
                    s0 = pair_sum<RL>(ph[0], ph[1], odd);     // H00 | H01
                    s1 = pair_sum<RL>(ph[2], ph[3], odd);     // H02 | H11
                    s2 = pair_sum<RL>(ph[4], ph[5], odd);     // H12 | H22
                    s3 = pair_sum<RL>(ph[6], ph[7], odd);     // b0  | b1
                    s4 = pair_sum<RL>(ph[8], pnv, odd);       // b2  | nv
                }
                // In a 4-lane surfel lanes 2 and 3 end with the sums of lanes 0
                // and 1, formed from the same two partial sums (the adds
                // commute), so they store the same words: no branch, and the
                // last butterfly add stays a DPP add over the whole wavefront.
                float* const o = lsm + (k * SLOTS + r) * SM_WORDS;
                if (LANES == 4 || p < (RL == 4 ? 4 : 2)) {
                    const int w = p & 1;
                    o[w] = s0; o[w + 2] = s1; o[w + 4] = s2; o[w + 6] = s3; o[w + 8] = s4;
                }
                if (with_cost) {
                    const float cs = group_sum<RL>(pcs);       // 4 lanes: the same in each
                    if (LANES == 4 || p < (RL == 4 ? 4 : 1)) o[SM_COST] = cs;
                }
            }
            wave_sync();
            // the owner's state and tangent basis, read back from the words it
            // wrote before the group loop rather than held in registers
            // through the frame loops
            __asm__ volatile("" ::: "memory");
            if (owner) {
                const float* o = lst + own * ST_WORDS;
                const float4 w0 = *(const float4*)(o + 0);
                const float4 w1 = *(const float4*)(o + 4);
                const float4 w2 = *(const float4*)(o + 8);
                const float4 w3 = *(const float4*)(o + 12);
                const float4 w4 = *(const float4*)(o + 16);
                id = w0.x; nx = w0.y; ny = w0.z; nz = w0.w;
                b1x = w1.x; b1y = w1.y; b1z = w1.z; b2x = w1.w; b2y = w2.x; b2z = w2.y;
                alive = w3.y != 0.f;
                flags = __float_as_uint(w3.z); lam = w3.w;
                cost_out = w4.x; nv_out = __float_as_int(w4.y);
            }
            // ---- owners: solve, update (Levenberg-Marquardt candidate test below)
            bool cand = false;
            float id_c = 0.f, nx_c = 0.f, ny_c = 0.f, nz_c = 0.f, cost_here = 0.f;
            int nv = 0;
            if (owner) {
                // The step of owner_step, written out here: as a call (forced
                // inline) the compiler allocates 5-10 more VGPRs for this
                // kernel, which spills in the default plan and costs the
                // one-group plans their sixth wavefront per SIMD.  The text
                // between the markers must equal owner_step's body; a CPU test
                // compares the two.  kappa^2 is formed here, each iteration,
                // rather than held in a register through the frame loops.
                float kappa_it = kappa_s;
                __asm__ volatile("" : "+s"(kappa_it));
                const float kap2 = kappa_it * kappa_it;
                // owner_step body begin
                const float* sm = lsm + own * SM_WORDS;
                const float H00 = sm[SM_H00], H01 = sm[SM_H01], H02 = sm[SM_H02];
                const float H11 = sm[SM_H11], H12 = sm[SM_H12], H22 = sm[SM_H22];
                const float bb0 = sm[SM_B0], bb1 = sm[SM_B1], bb2 = sm[SM_B2];
                nv = (int)sm[SM_NV];
                cost_here = sm[SM_COST];
                if (alive && last) cost_out = cost_here;
                if (alive) {
                    nv_out = nv;
                    float d0s = 0.f, d1s = 0.f, d2s = 0.f;
                    bool ok = true;
                    if (nv < 3) {
                        flags |= F_FEW_SAMPLES;
                        ok = false;
                    }
                    const float dd = 1.f + lam;          // (H + lam diag H): equilibrated diagonal
                    if (ok && depth_only) {
                        if (H00 > 0.f && isfinite(H00)) {
                            d0s = -bb0 * rcp_fast(H00 * dd);
                        } else {
                            flags |= F_SOLVE_FAIL;
                            ok = false;
                        }
                    } else if (ok) {
                        // equilibrate: E = D^-1/2 H D^-1/2 (unit diagonal).  The float
                        // solve is formed unconditionally (no branches: the tests below
                        // are combined with |) and replaced by the double-precision one
                        // where a diagonal is not positive and finite or the system is
                        // too ill-conditioned for float.
                        const float maxd = fmaxf(H00, fmaxf(H11, H22));
                        const float e0 = __frsqrt_rn(H00), e1 = __frsqrt_rn(H11), e2 = __frsqrt_rn(H22);
                        const float e01 = H01 * e0 * e1, e02 = H02 * e0 * e2, e12 = H12 * e1 * e2;
                        // adjugate and determinant of E (diagonal dd = 1 + lambda)
                        const float d2 = dd * dd;
                        const float c00 = fmaf(-e12, e12, d2), c11 = fmaf(-e02, e02, d2);
                        const float c22 = fmaf(-e01, e01, d2);
                        const float c01 = fmaf(e02, e12, -dd * e01), c02 = fmaf(e01, e12, -dd * e02);
                        const float c12 = fmaf(e01, e02, -dd * e12);
                        const float det = fmaf(e01, c01, fmaf(e02, c02, dd * c00));
                        // kappa_F(E)^2 = ||E||_F^2 ||adj E||_F^2 / det^2  (>= kappa_2(E)^2)
                        const float fro2 = 3.f * d2 + 2.f * (e01 * e01 + e02 * e02 + e12 * e12);
                        const float adj2 = c00 * c00 + c11 * c11 + c22 * c22 +
                                           2.f * (c01 * c01 + c02 * c02 + c12 * c12);
                        // raw Cholesky pivots are H_jj times the equilibrated ones
                        const float p1 = c22 * rcp_fast(dd);   // dd - e01^2 / dd (only compared)
                        const float p2 = det * rcp_fast(c22);  // (only compared)
                        const bool need64 = !(H00 > 0.f) | !(H11 > 0.f) | !(H22 > 0.f) | !isfinite(maxd) |
                                            !(fro2 * adj2 <= kap2 * det * det) | !(det > 0.f) | !(c22 > 0.f) |
                                            !(H11 * p1 > 1e-10f * maxd * dd) | !(H22 * p2 > 1e-10f * maxd * dd);
                        {
                            const float bh0 = bb0 * e0, bh1 = bb1 * e1, bh2 = bb2 * e2;
                            const float idet = rcp_fast(det);
                            d0s = -(c00 * bh0 + c01 * bh1 + c02 * bh2) * idet * e0;
                            d1s = -(c01 * bh0 + c11 * bh1 + c12 * bh2) * idet * e1;
                            d2s = -(c02 * bh0 + c12 * bh1 + c22 * bh2) * idet * e2;
                        }
                        if (need64) {
                            flags |= F_FP64_SOLVE;
                            double dd0 = 0.0, dd1 = 0.0, dd2 = 0.0;
                            const double dmp = 1.0 + (double)lam;
                            if (solve3_fp64((double)H00 * dmp, H01, H02, (double)H11 * dmp, H12,
                                            (double)H22 * dmp, bb0, bb1, bb2, dd0, dd1, dd2)) {
                                d0s = (float)dd0; d1s = (float)dd1; d2s = (float)dd2;
                            } else {
                                flags |= F_SOLVE_FAIL;
                                ok = false;
                            }
                        }
                    }
                    if (ok) {
                        // update: id_s += d0; n = normalise(n + d1 b1 + d2 b2) (the
                        // depth-only ablation moves id_s alone and keeps n)
                        id_c = id + d0s;
                        nx_c = nx; ny_c = ny; nz_c = nz;
                        bool ok_step;
                        if (depth_only) {
                            ok_step = (id_c > 0.f) && isfinite(id_c);
                        } else {
                            const float mx = fmaf(d1s, b1x, fmaf(d2s, b2x, nx));
                            const float my = fmaf(d1s, b1y, fmaf(d2s, b2y, ny));
                            const float mz = fmaf(d1s, b1z, fmaf(d2s, b2z, nz));
                            const float l2 = mx * mx + my * my + mz * mz;
                            ok_step = (id_c > 0.f) && isfinite(id_c) && (l2 > 0.f) && isfinite(l2);
                            if (ok_step) {
                                const float il = __frsqrt_rn(l2);
                                nx_c = mx * il; ny_c = my * il; nz_c = mz * il;
                            }
                        }
                        if (!ok_step) {
                            flags |= F_REJECTED;
                            if (lm) lam *= 10.f;
                        } else {
                            cand = true;
                        }
                    }
                }
                // owner_step body end
            }
            if (lm) {
                // Levenberg-Marquardt: the candidate's cost over the pixels,
                // then the acceptance test (lm_accept)
                float inv_cc = 0.f;
                bool cand_ok = cand;
                if (owner && cand) {
                    const float cc = nx_c * rsx + ny_c * rsy + nz_c;
                    if (fabsf(cc) < 1e-6f) {             // candidate plane contains r_s
                        flags |= F_REJECTED;
                        lam *= 10.f;
                        cand_ok = false;
                    }
                    inv_cc = rcp_fast(cc);
                }
                if (owner) {
                    float* o = lst + own * ST_WORDS;
                    o[ST_ID] = id_c; o[ST_NX] = nx_c; o[ST_NY] = ny_c; o[ST_NZ] = nz_c;
                    o[ST_INVC] = inv_cc;
                    o[ST_ALIVE] = cand_ok ? 1.f : 0.f;
                }
                wave_sync();
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const float* st = lst + (k * SLOTS + r) * ST_WORDS;
                    const float4 sa = *(const float4*)(st + 0);
                    const float inv_c = st[ST_INVC];
                    const bool calive = st[ST_ALIVE] != 0.f;
                    const int tx = it0x + (k % G.gx) * TX + r % TX, ty = it0y + (k / G.gx) * TY + r / TX;
                    float cst2 = 0.f;
                    int nv2l = 0;
                    const float cnx = sa.y * inv_c, cny = sa.z * inv_c;
                    const float sig0 = fmaf(cny, dry0, cnx * drx0);
                    const float dsig = cny * dyr_f;
                    if constexpr (SPLIT > 1) {
                        const float bdx = (float)(S * tx + pxs[0] - bpx) - 0.5f * (float)(G.ab * S - 1);
                        float bdy[PPL], idu_c[PPL];
                        bool pok[PPL];
#pragma unroll
                        for (int j = 0; j < PPL; ++j) {
                            const int row = row0 + SPLIT * j;
                            const float sig = row == 0 ? sig0 : fmaf((float)row, dsig, sig0);
                            idu_c[j] = fmaf(sa.x, sig, sa.x);
                            bdy[j] = (float)(S * ty + pys[j] - bpy) - 0.5f * (float)(G.ab * S - 1);
                            pok[j] = calive && (idu_c[j] > 0.f);
                        }
                        split_cost<T, BY_ROW, PPL, SPLIT>(pairs, fr, nf, bdx, bdy, idu_c, pok, pitch_b, wm1, hm1,
                                                          ikf[k], hk, img_scale, row0, s_terms[wave] + lane, cst2,
                                                          nv2l);
                    }
#pragma unroll
                    for (int j = 0; SPLIT == 1 && j < PPL; ++j) {
                        const float sig = j == 0 ? sig0 : fmaf((float)j, dsig, sig0);
                        const float idu_c = fmaf(sa.x, sig, sa.x);
                        float bdx = (float)(S * tx + pxs[j] - bpx) - 0.5f * (float)(G.ab * S - 1);
                        float bdy = (float)(S * ty + pys[j] - bpy) - 0.5f * (float)(G.ab * S - 1);
                        // formed here, not kept from the item's start through the
                        // iterations (registers)
                        __asm__ volatile("" : "+v"(bdx), "+v"(bdy));
                        frame_cost<T, BY_ROW, DEEP ? 4 : 0>(pairs, fr, nf, bdx, bdy, idu_c, calive && (idu_c > 0.f),
                                                           pitch_b, wm1, hm1, ikf[k][j], hk, img_scale, cst2, nv2l);
                    }
                    // (a split column's cost stands in its last row's lanes)
                    const float c2 = group_sum<RL>(cst2);
                    const int n2 = group_sum<LANES>(nv2l);
                    if (p == LANES - RL) {
                        float* o = lsm + (k * SLOTS + r) * SM_WORDS;
                        o[SM_COST] = c2;
                        o[SM_NV] = __int_as_float(n2);
                    }
                }
                wave_sync();
                if (owner && cand_ok) {
                    const float* sm = lsm + own * SM_WORDS;
                    cand_ok = lm_accept(sm[SM_COST], __float_as_int(sm[SM_NV]), cost_here, nv, lam);
                }
                cand = cand_ok;
            }
            if (owner && cand) {
                id = id_c;
                nx = nx_c; ny = ny_c; nz = nz_c;
                updated = true;
            }
        }
        if (own_ok) {
            ((gmut<float>)Kd->inv_depth)[sidx] = id;
            ((gmut<float>)Kd->nx)[sidx] = nx;
            ((gmut<float>)Kd->ny)[sidx] = ny;
            ((gmut<float>)Kd->nz)[sidx] = nz;
            ((gmut<uint32_t>)Kd->flags)[sidx] = flags;
            ((gmut<float>)Kd->cost)[sidx] = iters > 0 ? cost_out : 0.f;
            ((gmut<uint32_t>)Kd->nvalid)[sidx] = (uint32_t)(iters > 0 ? nv_out : 0);
            if (updated) ((gmut<uint32_t>)Kd->last_update)[sidx] = stamp;
        }
    }
}

// Where a workgroup shares its surfels' solves, a surfel's state lives in its
// ST_ words.  Degeneracy and tangent basis, before each iteration (n . r_s
// with the roundings that gn_kernel and disc_gn_kernel give it):
template <bool DISC>
__device__ __forceinline__ void surfel_ready(float* o, float nx, float ny, float nz, bool alive, uint32_t flags) {
    const float rx = o[ST_RSX], ry = o[ST_RSY];
    const float c = (DISC ? fmaf(ny, ry, nx * rx) : fmaf(nx, rx, ny * ry)) + nz;
    if (alive && fabsf(c) < 1e-6f) {
        o[ST_FLAGS] = __uint_as_float(flags | F_DEGENERATE);
        o[ST_ALIVE] = 0.f;
        o[ST_COSTO] = 0.f;
        o[ST_NVO] = __int_as_float(0);
    }
    float b1x, b1y, b1z, b2x, b2y, b2z;
    tangent_basis(nx, ny, nz, b1x, b1y, b1z, b2x, b2y, b2z);
    o[ST_B1X] = b1x; o[ST_B1Y] = b1y; o[ST_B1Z] = b1z;
    o[ST_B2X] = b2x; o[ST_B2Y] = b2y; o[ST_B2Z] = b2z;
    o[ST_INVC] = rcp_fast(c);
}
// and the undamped step from its sums, the next iteration's basis included.
template <bool DISC>
__device__ __forceinline__ void shared_step(float* o, const float* sm, bool last, bool depth_only, float kap2) {
    const float4 w0 = *(const float4*)(o + 0);
    const float4 w1 = *(const float4*)(o + 4);
    const float4 w2 = *(const float4*)(o + 8);
    const float4 w3 = *(const float4*)(o + 12);
    const float4 w4 = *(const float4*)(o + 16);
    const bool alive = w3.y != 0.f;
    if (!alive) return;
    uint32_t flags = __float_as_uint(w3.z);
    float cost_out = w4.x, cost_here = 0.f, id_c = 0.f, nx_c = 0.f, ny_c = 0.f, nz_c = 0.f, lam = 0.f;
    int nv_out = __float_as_int(w4.y), nv = 0;
    const bool step = owner_step(sm, alive, last, depth_only, false, kap2, lam, w0.x, w0.y, w0.z, w0.w, w1.x, w1.y,
                                 w1.z, w1.w, w2.x, w2.y, flags, cost_out, nv_out, nv, cost_here, id_c, nx_c, ny_c,
                                 nz_c);
    o[ST_FLAGS] = __uint_as_float(flags);
    o[ST_COSTO] = cost_out; o[ST_NVO] = __int_as_float(nv_out);
    if (step) {
        o[ST_ID] = id_c; o[ST_NX] = nx_c; o[ST_NY] = ny_c; o[ST_NZ] = nz_c;
        o[ST_LAM] = 1.f;
    }
    if (!last) surfel_ready<DISC>(o, step ? nx_c : w0.y, step ? ny_c : w0.z, step ? nz_c : w0.w, true, flags);
}

// The Gauss-Newton kernel of large grids: gn_kernel without damping, four
// pixels per lane, one group per wavefront, whose workgroup shares its
// surfels' solves.  After each iteration's sums one wavefront (another each
// time) steps the surfels of all four items, a lane each, between two
// barriers; in gn_kernel every wavefront issues the step with most of its
// lanes idle.  The arithmetic and the order of every sum are gn_kernel's.
//
// Bound: VALU issue.  The step is about 170 of the 1,450 instructions that a
// wavefront of sixteen 4x4 surfels issues per iteration at seven neighbour
// frames (more for one 16 x 16 surfel), and three quarters of it goes; with
// the surfels' state in LDS and no damped branch the rest also takes fewer
// registers: eight wavefronts per SIMD (64 VGPRs) one sample at a time, six
// (80) with a frame's taps in flight, where gn_kernel held seven and five.
// 64 mixed keyframes: f16 4.15 -> 3.77 ms, f32 4.13 -> 3.93, u8 4.12 -> 3.86;
// 1920x1080 f16 415 -> 391 us.  (At the old seven and five: 4.07, 4.00 and
// 3.91 ms.  Raising the stepping wavefront's priority gave nothing.)
template <typename T, int S, int TX, int TY, bool BY_ROW, int DEEP>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(DEEP ? 6 : 8, 8))) void gn_shared_kernel(
    LoneBatch, const BatchHeader* __restrict__ hdr_) {
    constexpr ItemGeo G = item_geo(S, TX, TY, 1);
    constexpr int PIX = S * S;
    constexpr int NS = TX * TY;                               // surfels per work item
    constexpr int LANES = kWaveSize / NS;
    constexpr int PPL = PIX / LANES;
    constexpr float DYR = (float)(LANES / S);
    constexpr int WPB = kBlockThreads / kWaveSize;
    static_assert(PPL == 4 && WPB * NS <= kWaveSize, "four pixels per lane; a lane per surfel of the workgroup");
    const BatchView view = batch_view(hdr_);
    const cptr<BatchHeader> hdr = view.hdr;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane / LANES;
    const int p = lane % LANES;
    const float half = 0.5f * (float)(S - 1);
    const int px0 = p % S, py0 = p / S;
    constexpr int DROW = LANES / S;

    __shared__ float4 s_pairs[WPB][kMaxNbr * kPairWords / 4];
    __shared__ float4 s_state[WPB * NS * ST_WORDS / 4];
    __shared__ float4 s_sums[WPB * NS * SM_WORDS / 4];
    float* const pairs = (float*)s_pairs[wave];
    float* const lst = (float*)s_state + wave * NS * ST_WORDS;
    float* const lsm = (float*)s_sums + wave * NS * SM_WORDS;

    const int total = hdr->total_items;
    const int iters = hdr->iters;
    const cptr<KfDev> kfs = view.kfs;
    // the workgroup's first item (see gn_kernel for the XCD shares)
    int first = (int)blockIdx.x * WPB, end = total;
    if (hdr->n_queues == kXcds) {
        const int share = (int)(blockIdx.x % (unsigned)kXcds);
        first = hdr->queues[share].begin + (int)(blockIdx.x / (unsigned)kXcds) * WPB;
        end = hdr->queues[share].end;
    }
    if (first >= end) return;                                 // the whole workgroup
    const int item = first + wave;
    // a wavefront without an item keeps to the workgroup's barriers
    int it0x = 0, it0y = 0;
    bool work = item < end;
    cptr<KfDev> Kd = kfs;
    int bx = 0, by = 0;
    if (work) {
        Kd = kfs + find_kf(kfs, hdr->n_kf, item, 0);
        const int blk = item - Kd->item_base;                 // one item per anchor block
        static_assert(G.ipb == 1, "an item is an anchor block");
        bx = blk % Kd->groups_x; by = blk / Kd->groups_x;
        it0x = bx * G.ab; it0y = by * G.ab;
        work = it0x < Kd->gw && it0y < Kd->gh;
    }
    const int gw = Kd->gw, gh = Kd->gh;
    const int nf = Kd->n_nbr;
    const float img_scale = Kd->img_scale;
    const unsigned pitch_b = (unsigned)Kd->nbr_pitch_b;
    const unsigned wm1 = (unsigned)(Kd->width - 1), hm1 = (unsigned)(Kd->height - 1);
    const float fxk = Kd->fx, fyk = Kd->fy, cxk = Kd->cx, cyk = Kd->cy;
    const float drx0 = ((float)px0 - half) / fxk, dry0 = ((float)py0 - half) / fyk;
    const float dyr_f = DYR / fyk;
    const int bpx = bx * G.ab * S, bpy = by * G.ab * S;
    if (work)
        stage_pair_words(view.frames + Kd->frame_base, nf, lane, (double)bpx + 0.5 * (double)(G.ab * S - 1),
                         (double)bpy + 0.5 * (double)(G.ab * S - 1), pairs);
    const uint64_t fr_bits = (uint64_t)(view.frames + Kd->frame_base);
    const uint32_t fr_lo = __builtin_amdgcn_readfirstlane((uint32_t)fr_bits);
    const uint32_t fr_hi = __builtin_amdgcn_readfirstlane((uint32_t)(fr_bits >> 32));
    const cptr<FrameDev> fr = (cptr<FrameDev>)(((uint64_t)fr_hi << 32) | fr_lo);
    const int tx = it0x + r % TX, ty = it0y + r / TX;
    float ikf[PPL];
    const gptr<T> kimg = (gptr<T>)Kd->kf_img;
#pragma unroll
    for (int j = 0; j < PPL; ++j) {
        ikf[j] = 0.f;
        if (work && tx < gw && ty < gh)
            ikf[j] = ldg<T>(kimg + ((unsigned)(S * ty + py0 + DROW * j) * (unsigned)Kd->kf_pitch +
                                    (unsigned)(S * tx + px0))) * Kd->kf_scale;
    }
    // this item's surfels, lane k < NS the k-th
    const int otx = it0x + lane % TX, oty = it0y + lane / TX;
    const bool own_ok = work && lane < NS && otx < gw && oty < gh;
    const int sidx = oty * gw + otx;
    if (lane < NS) {
        float* o = lst + lane * ST_WORDS;
        o[ST_ID] = own_ok ? ((gptr<float>)Kd->inv_depth)[sidx] : 0.f;
        o[ST_NX] = own_ok ? ((gptr<float>)Kd->nx)[sidx] : 0.f;
        o[ST_NY] = own_ok ? ((gptr<float>)Kd->ny)[sidx] : 0.f;
        o[ST_NZ] = own_ok ? ((gptr<float>)Kd->nz)[sidx] : -1.f;
        const float usx = (float)(S * otx) + half, usy = (float)(S * oty) + half;
        o[ST_RSX] = (usx - cxk) / fxk; o[ST_RSY] = (usy - cyk) / fyk;
        o[ST_ALIVE] = own_ok ? 1.f : 0.f;
        o[ST_FLAGS] = __uint_as_float(own_ok ? ((gptr<uint32_t>)Kd->flags)[sidx] & ~F_GN_BITS : 0u);
        o[ST_LAM] = 0.f;                                      // set once a step is accepted
        o[ST_COSTO] = 0.f; o[ST_NVO] = __int_as_float(0);
    }
    wave_sync();
    if (iters > 0 && lane < NS) {
        float* o = lst + lane * ST_WORDS;
        surfel_ready<false>(o, o[ST_NX], o[ST_NY], o[ST_NZ], o[ST_ALIVE] != 0.f, __float_as_uint(o[ST_FLAGS]));
    }
    wave_sync();
    for (int it = 0; it < iters; ++it) {
        const bool last = it == iters - 1;
        if (work) {
            const float* st = lst + r * ST_WORDS;
            float ph[9], pnv, pcs;
            {
                const float4 sa = *(const float4*)(st + 0);      // id, nx, ny, nz
                const float sid = sa.x, snx = sa.y, sny = sa.z;
                const float inv_c = st[ST_INVC];
                const bool salive = st[ST_ALIVE] != 0.f;
                bool pix_ok[PPL];
                const float cnx = snx * inv_c, cny = sny * inv_c;
                const float sig0 = fmaf(cny, dry0, cnx * drx0);
                const float dsig = cny * dyr_f;
                const float idu0 = fmaf(sid, sig0, sid);
                const float didu = sid * dsig;
#pragma unroll
                for (int j = 0; j < PPL; ++j) {
                    const float sig = j == 0 ? sig0 : fmaf((float)j, dsig, sig0);
                    pix_ok[j] = salive && (fmaf(sid, sig, sid) > 0.f);
                }
                const float bdx = (float)(S * tx + px0 - bpx) - 0.5f * (float)(G.ab * S - 1);
                const float bdy = (float)(S * ty + py0 - bpy) - 0.5f * (float)(G.ab * S - 1);
                float A[PPL], B[PPL], cst[PPL];
                unsigned nvp = 0u;
#pragma unroll
                for (int j = 0; j < PPL; ++j) {
                    A[j] = 0.f; B[j] = 0.f; cst[j] = 0.f;
                }
                const float hk = hdr->huber_k;
                if (last)
                    frame_loop_px<T, true, PPL, BY_ROW, DEEP, 1>(pairs, fr, nf, bdx, bdy, DYR, idu0, didu, 0, pix_ok,
                                                                 pitch_b, wm1, hm1, ikf, hk, img_scale, A, B, cst, nvp);
                else
                    frame_loop_px<T, false, PPL, BY_ROW, DEEP, 1>(pairs, fr, nf, bdx, bdy, DYR, idu0, didu, 0, pix_ok,
                                                                  pitch_b, wm1, hm1, ikf, hk, img_scale, A, B, cst, nvp);
                __asm__ volatile("" ::: "memory");
                const float4 sa2 = *(const float4*)(st + 0);
                const float4 sb = *(const float4*)(st + 4);
                const float4 sc = *(const float4*)(st + 8);
                const float srsy = st[ST_RSY];
                const float sb1x = sb.x, sb1y = sb.y, sb1z = sb.z;
                const float sb2x = sb.w, sb2y = sc.x, sb2z = sc.y, srsx = sc.w;
                const float pinv_c = sc.z;
                const float pcnx = sa2.y * pinv_c, pcny = sa2.z * pinv_c;
                const float psig0 = fmaf(pcny, dry0, pcnx * drx0);
                const float pdsig = pcny * dyr_f;
                const float kk = hdr->depth_only != 0 ? 0.f : sa2.x * pinv_c;
                const float k1x = kk * sb1x, k1y = kk * sb1y, k2x = kk * sb2x, k2y = kk * sb2y;
                const float q1 = kk * fmaf(sb1x, srsx, fmaf(sb1y, srsy, sb1z));
                const float q2 = kk * fmaf(sb2x, srsx, fmaf(sb2y, srsy, sb2z));
                const float g00 = 1.f + psig0;
                const float g10 = fmaf(-psig0, q1, fmaf(k1y, dry0, k1x * drx0));
                const float g20 = fmaf(-psig0, q2, fmaf(k2y, dry0, k2x * drx0));
                const float dg1 = fmaf(-pdsig, q1, k1y * dyr_f);
                const float dg2 = fmaf(-pdsig, q2, k2y * dyr_f);
                const float S0 = (A[0] + A[1]) + (A[2] + A[3]);
                const float S1 = fmaf(3.f, A[3], fmaf(2.f, A[2], A[1]));
                const float S2 = fmaf(9.f, A[3], fmaf(4.f, A[2], A[1]));
                const float T0 = (B[0] + B[1]) + (B[2] + B[3]);
                const float T1 = fmaf(3.f, B[3], fmaf(2.f, B[2], B[1]));
                const float ga[3] = {g00, g10, g20}, gb[3] = {pdsig, dg1, dg2};
                float uu[3], vv[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    uu[a] = fmaf(S1, gb[a], S0 * ga[a]);
                    vv[a] = fmaf(S2, gb[a], S1 * ga[a]);
                }
                ph[0] = fmaf(vv[0], gb[0], uu[0] * ga[0]);
                ph[1] = fmaf(vv[0], gb[1], uu[0] * ga[1]);
                ph[2] = fmaf(vv[0], gb[2], uu[0] * ga[2]);
                ph[3] = fmaf(vv[1], gb[1], uu[1] * ga[1]);
                ph[4] = fmaf(vv[1], gb[2], uu[1] * ga[2]);
                ph[5] = fmaf(vv[2], gb[2], uu[2] * ga[2]);
#pragma unroll
                for (int a = 0; a < 3; ++a) ph[6 + a] = fmaf(T1, gb[a], T0 * ga[a]);
                pcs = (cst[0] + cst[1]) + (cst[2] + cst[3]);
                pnv = (float)__builtin_amdgcn_sad_u8(nvp, 0u, 0u);
            }
            {
#pragma clang fp contract(off)
                const bool odd = (p & 1) != 0;
                const float s0 = pair_sum<LANES>(ph[0], ph[1], odd);
                const float s1 = pair_sum<LANES>(ph[2], ph[3], odd);
                const float s2 = pair_sum<LANES>(ph[4], ph[5], odd);
                const float s3 = pair_sum<LANES>(ph[6], ph[7], odd);
                const float s4 = pair_sum<LANES>(ph[8], pnv, odd);
                float* const o = lsm + r * SM_WORDS;
                if (LANES == 4 || p < 2) {
                    const int w = p & 1;
                    o[w] = s0; o[w + 2] = s1; o[w + 4] = s2; o[w + 6] = s3; o[w + 8] = s4;
                }
                if (last) {
                    const float cs = group_sum<LANES>(pcs);
                    if (LANES == 4 || p == 0) o[SM_COST] = cs;
                }
            }
        }
        __syncthreads();
        if (wave == (int)((blockIdx.x / kXcds + (unsigned)it) % WPB) && lane < WPB * NS) {
            const float kap = hdr->kappa_fp64;
            shared_step<false>((float*)s_state + lane * ST_WORDS, (const float*)s_sums + lane * SM_WORDS, last,
                               hdr->depth_only != 0, kap * kap);
        }
        __syncthreads();
    }
    if (own_ok) {
        const float* o = lst + lane * ST_WORDS;
        ((gmut<float>)Kd->inv_depth)[sidx] = o[ST_ID];
        ((gmut<float>)Kd->nx)[sidx] = o[ST_NX];
        ((gmut<float>)Kd->ny)[sidx] = o[ST_NY];
        ((gmut<float>)Kd->nz)[sidx] = o[ST_NZ];
        ((gmut<uint32_t>)Kd->flags)[sidx] = __float_as_uint(o[ST_FLAGS]);
        ((gmut<float>)Kd->cost)[sidx] = o[ST_COSTO];
        ((gmut<uint32_t>)Kd->nvalid)[sidx] = __float_as_uint(o[ST_NVO]);
        if (o[ST_LAM] != 0.f) ((gmut<uint32_t>)Kd->last_update)[sidx] = hdr->stamp;
    }
}

// ----------------------------------------------------------- render kernel --

// Inverse Depth Calculation section: each pixel takes Eq. 3 of its surfel,
// id_u = id_s (1 + sigma), sigma = n . (r_u - r_s) / (n . r_s).  A thread
// renders a block of 4 x 4 pixels, which lies in one tile (blocks past the
// grid write "no measurement"): the surfel's state is read once for four
// 16-byte row stores.  A wavefront takes 64 blocks of one keyframe, a row of
// them after the other, and reads the keyframe through scalar loads.
//
// Bound: the writes.  64 mixed keyframes (26.8 million pixels, 107 MB):
// 72 us with one row segment per thread, each workgroup searching its
// keyframe first and each thread reading the descriptor through vector
// loads; 31 us now, a copy's rate 21.
__global__ __launch_bounds__(256) void render_kernel(LoneKf, const BatchHeader* __restrict__ hdr_) {
#pragma clang fp contract(off)
    const BatchView view = batch_view(hdr_);
    const cptr<BatchHeader> hdr = view.hdr;
    const cptr<KfDev> kfs = view.kfs;
    const int lane = threadIdx.x & (kWaveSize - 1);
    for (int wv = grid_wave(); wv < hdr->render_waves; wv += grid_waves()) {
        // (keyframes without an output take no wavefront)
        int lo = 0, hi = hdr->n_kf - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (kfs[mid].render_wave <= wv) lo = mid; else hi = mid - 1;
        }
        const carg<KfDev>& K = kfs[lo];
        const int W = K.width, H = K.height, S = K.patch;
        const int nbx = (W + 3) / 4, nby = (H + 3) / 4;
        const int blk = (wv - K.render_wave) * kWaveSize + lane;
        if (blk >= nbx * nby) continue;
        const int by = divide(blk, K.div_bx), bx = blk - by * nbx;
        const int x0 = 4 * bx, y0 = 4 * by;
        const int sh = __builtin_ctz(S);                  // S is 4, 8 or 16
        const int tx = x0 >> sh, ty = y0 >> sh;
        const float half = 0.5f * (float)(S - 1);
        const float ifx = 1.f / K.fx, ify = 1.f / K.fy;
        bool ok = false;
        int i = -1;
        float id = 0.f, nx = 0.f, ny = 0.f, inv_c = 1.f, usx = 0.f, usy = 0.f;
        if (tx < K.gw && ty < K.gh) {
            i = ty * K.gw + tx;
            // the state is loaded with the flags (one round trip, not two);
            // a flagged surfel's values are not used
            const uint32_t fl = K.flags[i];
            const float snx = K.nx[i], sny = K.ny[i], snz = K.nz[i], sid = K.inv_depth[i];
            // (kept in front of the flag test, where the compiler would sink them)
            __asm__ volatile("" ::"v"(snx), "v"(sny), "v"(snz), "v"(sid));
            if (!(fl & (F_DEGENERATE | F_UNINIT))) {
                usx = (float)(S * tx) + half;
                usy = (float)(S * ty) + half;
                const float rsx = (usx - K.cx) * ifx, rsy = (usy - K.cy) * ify;
                nx = snx;
                ny = sny;
                const float c = fmaf(nx, rsx, ny * rsy) + snz;
                id = sid;
                ok = fabsf(c) >= 1e-6f;
                inv_c = 1.f / c;
            }
        }
        float drx[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) drx[j] = ((float)(x0 + j) - usx) * ifx;
        float* const out = K.inv_depth_out;
        int32_t* const idx_out = K.index_out;
        // whole aligned rows of four in one store: the same for every block
        // of the keyframe
        const bool rows4 = (W & 3) == 0 && ((uintptr_t)out & 15u) == 0 && ((uintptr_t)idx_out & 15u) == 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int y = y0 + r;
            if (y >= H) break;
            const float ndy = ny * (((float)y - usy) * ify);
            float v[4];
            int w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float sigma = fmaf(nx, drx[j], ndy) * inv_c;
                const float idu = fmaf(id, sigma, id);
                const bool hit = ok && idu > 0.f && isfinite(idu);
                v[j] = hit ? idu : 0.f;
                w[j] = hit ? i : -1;
            }
            const size_t o = (size_t)y * W + x0;
            if (rows4) {
                *(float4*)(out + o) = make_float4(v[0], v[1], v[2], v[3]);
                if (idx_out) *(int4*)(idx_out + o) = make_int4(w[0], w[1], w[2], w[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (x0 + j >= W) continue;
                    out[o + j] = v[j];
                    if (idx_out) idx_out[o + j] = w[j];
                }
            }
        }
    }
}

// ----------------------------------------------------------- regrid kernels --

// Surfel reference-frame change (Eq. 10) and re-gridding into the tiles of
// another keyframe.  Every landing decision (destination tile, closest
// surfel) is taken in double with a fixed operation order and no
// contraction, so it is the same decision the plain double definition takes.
struct Land {
    double idp, rp0, rp1, np0, np1, np2;
    int tile;
};

// (NORMAL: with the moved normal, which the landing does not depend on.)
template <bool NORMAL>
__device__ __forceinline__ bool regrid_land(const carg<RegridArgs>& a, int i, Land& L) {
#pragma clang fp contract(off)
    const int S0 = 1 << a.src_shift;
    const int ty = divide(i, a.div_src), tx = i - ty * a.src_gw;
    // every load before the first test: one round trip instead of three
    const uint32_t fl = a.src.flags[i];
    const float fid = a.src.inv_depth[i];
    float fn0 = 0.f, fn1 = 0.f, fn2 = 0.f;
    if constexpr (NORMAL) {
        fn0 = a.src.nx[i]; fn1 = a.src.ny[i]; fn2 = a.src.nz[i];
        __asm__ volatile("" ::"v"(fn0), "v"(fn1), "v"(fn2));
    }
    __asm__ volatile("" ::"v"(fl), "v"(fid));
    if (fl & (F_DEGENERATE | F_UNINIT)) return false;
    const double id = (double)fid;
    if (!(id > 0.0) || !isfinite(id)) return false;
    const double usx = S0 * tx + 0.5 * (S0 - 1), usy = S0 * ty + 0.5 * (S0 - 1);
    const double rs0 = (usx - a.src_K[2]) / a.src_K[0], rs1 = (usy - a.src_K[3]) / a.src_K[1];
    const double p00 = rs0 / id, p01 = rs1 / id, p02 = 1.0 / id;          // Eq. 1
    const double n0 = fn0, n1 = fn1, n2 = fn2;
    const cptr<double> R = a.R;
    const double p10 = R[0] * p00 + R[1] * p01 + R[2] * p02 + a.t[0];
    const double p11 = R[3] * p00 + R[4] * p01 + R[5] * p02 + a.t[1];
    const double p12 = R[6] * p00 + R[7] * p01 + R[8] * p02 + a.t[2];
    if constexpr (NORMAL) {
        L.np0 = R[0] * n0 + R[1] * n1 + R[2] * n2;
        L.np1 = R[3] * n0 + R[4] * n1 + R[5] * n2;
        L.np2 = R[6] * n0 + R[7] * n1 + R[8] * n2;
    }
    if (!(p12 > 0.0)) return false;
    L.rp0 = p10 / p12;
    L.rp1 = p11 / p12;
    const double ux = a.dst_K[0] * L.rp0 + a.dst_K[2], uy = a.dst_K[1] * L.rp1 + a.dst_K[3];
    const double px = floor(ux + 0.5), py = floor(uy + 0.5);          // nearest pixel
    const int sh = a.dst_shift;
    if (!(px >= 0.0 && px < (double)(a.dst_gw << sh) && py >= 0.0 && py < (double)(a.dst_gh << sh))) return false;
    L.tile = ((int)py >> sh) * a.dst_gw + ((int)px >> sh);
    L.idp = 1.0 / p12;
    return true;
}

// The re-gridding kernels run over a table of keyframe pairs in wavefronts
// of 64 lanes that never span two pairs: pair k's sources (destination
// tiles) take the wavefronts from src_wave (dst_wave) on, so the entry is
// the last whose first wavefront is <= the wavefront's number.  It is found
// and read with wavefront-uniform (scalar) loads.
template <bool DST>
__device__ __forceinline__ int regrid_entry_of_wave(cptr<RegridArgs> tab, int n, int wv) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((DST ? tab[mid].dst_wave : tab[mid].src_wave) <= wv) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Clears the landing keys and winners of all the batch's tiles (n_tiles of
// each) and brings the table up, in one launch: workgroups past the table's
// words fill, 16 bytes per thread and store.
__global__ __launch_bounds__(256) void regrid_clear_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst,
                                                           int n16, uint4* __restrict__ best, int nb16,
                                                           uint4* __restrict__ win, int nw16) {
    const int copy_blocks = (n16 + 255) / 256;
    if ((int)blockIdx.x < copy_blocks) {
        const int i = (int)(blockIdx.x * 256 + threadIdx.x);
        if (i < n16) dst[i] = src[i];
        return;
    }
    const int step = (int)(gridDim.x - copy_blocks) * 256;
    const int i0 = (int)((blockIdx.x - copy_blocks) * 256 + threadIdx.x);
    for (int i = i0; i < nb16; i += step) best[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int i = i0; i < nw16; i += step) win[i] = make_uint4(0x7fffffffu, 0x7fffffffu, 0x7fffffffu, 0x7fffffffu);
}

// pass 0: closest landing per tile (1/p'_z > 0, so its bits order like the
// value); pass 1: the lowest source index among the closest
__global__ __launch_bounds__(256) void regrid_scatter_kernel(RegridArgs, const RegridArgs* __restrict__ tab_, int n_pairs,
                                                             int src_waves, int pass) {
    const cptr<RegridArgs> tab = table_or_arg(tab_);
    const int lane = threadIdx.x & 63;
    for (int wv = grid_wave(); wv < src_waves; wv += grid_waves()) {
        const carg<RegridArgs>& a = tab[regrid_entry_of_wave<false>(tab, n_pairs, wv)];
        const int i = (wv - a.src_wave) * 64 + lane;
        Land L;
        if (i >= a.src_count || !regrid_land<false>(a, i, L)) continue;
        const unsigned long long bits = (unsigned long long)__double_as_longlong(L.idp);
        if (pass == 0)
            atomicMax(&a.best[L.tile], bits);
        else if (a.best[L.tile] == bits)
            atomicMin(&a.win[L.tile], i);
    }
}

__global__ __launch_bounds__(256) void regrid_gather_kernel(RegridArgs, const RegridArgs* __restrict__ tab_, int n_pairs,
                                                            int dst_waves) {
#pragma clang fp contract(off)
    const cptr<RegridArgs> tab = table_or_arg(tab_);
    const int lane = threadIdx.x & 63;
    for (int wv = grid_wave(); wv < dst_waves; wv += grid_waves()) {
        const carg<RegridArgs>& a = tab[regrid_entry_of_wave<true>(tab, n_pairs, wv)];
        const int j = (wv - a.dst_wave) * 64 + lane;
        if (j >= a.dst_count) continue;
        const int S1 = 1 << a.dst_shift;
        const int ty = divide(j, a.div_dst), tx = j - ty * a.dst_gw;
        const int w = a.win[j];
        // (loaded with the winner's state, not after it)
        const uint32_t stamp = w != 0x7fffffff ? a.src.last_update[w] : 0u;
        bool ok = false;
        double idt = 0.0, t0 = 0.0, t1 = 0.0, t2 = -1.0;
        Land L;
        if (w != 0x7fffffff && regrid_land<true>(a, w, L)) {
            const double rt0 = (S1 * tx + 0.5 * (S1 - 1) - a.dst_K[2]) / a.dst_K[0];
            const double rt1 = (S1 * ty + 0.5 * (S1 - 1) - a.dst_K[3]) / a.dst_K[1];
            const double c1 = L.np0 * L.rp0 + L.np1 * L.rp1 + L.np2 * 1.0;
            const double ct = L.np0 * rt0 + L.np1 * rt1 + L.np2 * 1.0;
            if (fabs(c1) >= 1e-6 && fabs(ct) >= 1e-6) {
                idt = L.idp * ct / c1;                    // Eq. 3 of the moved plane at r_t
                const double l = sqrt(L.np0 * L.np0 + L.np1 * L.np1 + L.np2 * L.np2);
                if (idt > 0.0 && isfinite(idt) && l > 0.0 && isfinite(l)) {
                    t0 = L.np0 / l; t1 = L.np1 / l; t2 = L.np2 / l;
                    ok = true;
                }
            }
        }
        a.dst.inv_depth[j] = ok ? (float)idt : 0.f;
        a.dst.nx[j] = ok ? (float)t0 : 0.f;
        a.dst.ny[j] = ok ? (float)t1 : 0.f;
        a.dst.nz[j] = ok ? (float)t2 : -1.f;
        a.dst.flags[j] = ok ? 0u : F_UNINIT;
        a.dst.cost[j] = 0.f;
        a.dst.nvalid[j] = 0u;
        a.dst.last_update[j] = ok ? stamp : 0u;
        a.is_new[j] = ok ? 0 : 1;
        if (a.src_index) a.src_index[j] = ok ? w : -1;
    }
}

hipError_t launch_regrid(const RegridArgs& one, const void* host, RegridArgs* table, size_t table_bytes,
                         int n_pairs, int src_waves, int dst_waves, void* best, void* win, int n_tiles,
                         hipStream_t s, hipEvent_t uploaded) {
    // four wavefronts per workgroup
    auto blocks = [](int waves) { return std::max(1, std::min(65536, (waves + 3) / 4)); };
    const int n16 = (int)((table_bytes + 15) / 16);
    // (the scratch arrays are padded to 256 bytes)
    const int nb16 = (int)(((size_t)n_tiles * 8 + 15) / 16), nw16 = (int)(((size_t)n_tiles * 4 + 15) / 16);
    const int fill = std::max(1, std::min(4096, (nb16 + 255) / 256));
    hipLaunchKernelGGL(regrid_clear_kernel, dim3((n16 + 255) / 256 + fill), dim3(256), 0, s, (const uint4*)host,
                       (uint4*)table, n16, (uint4*)best, nb16, (uint4*)win, nw16);
    if (uploaded) {
        const hipError_t e = hipEventRecord(uploaded, s);
        if (e != hipSuccess) return e;
    }
    if (src_waves > 0) {
        hipLaunchKernelGGL(regrid_scatter_kernel, dim3(blocks(src_waves)), dim3(256), 0, s, one, table, n_pairs,
                           src_waves, 0);
        hipLaunchKernelGGL(regrid_scatter_kernel, dim3(blocks(src_waves)), dim3(256), 0, s, one, table, n_pairs,
                           src_waves, 1);
    }
    hipLaunchKernelGGL(regrid_gather_kernel, dim3(blocks(dst_waves)), dim3(256), 0, s, one, table, n_pairs,
                       dst_waves);
    return hipGetLastError();
}

// --------------------------------------------------------- quantize kernel --

// One stored value of a sampled one.
__device__ __forceinline__ _Float16 stored_f16(float v, float scale) { return (_Float16)(v / scale); }
__device__ __forceinline__ uint8_t stored_u8(float v, float scale) {
    return (uint8_t)fminf(fmaxf(rintf(v / scale), 0.f), 255.f);
}

// f32 images to f16 or u8, eight pixels of a row per thread.  Where every row
// starts on 16 bytes of the source and 16 (f16) or 8 (u8) of the destination
// (VEC) they are neighbours, two 16-byte loads and one store; else they lie 64
// apart, so that the wavefront's loads and stores join up.  Bound: memory;
// 1920x1080 to f16 moves 12.4 MB.  One pixel per thread, its row found by a
// 64-bit division, took 5.2 us a call back to back, 15.3 at 3840x2160; VEC
// 4.1 and 8.7.  Rows that allow no wide loads: 4095x2159 to f16 16.5 us with a
// pixel per thread, 26.2 with eight neighbours, 11.1 now.
template <int DTYPE, bool VEC>
__global__ __launch_bounds__(256) void quantize_kernel(const float* __restrict__ src, int src_pitch,
                                                       void* __restrict__ dst, int dst_pitch, int width, int height,
                                                       float scale) {
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int x0 = 8 * kWaveSize * (int)blockIdx.x + (VEC ? 8 * lane : lane);
    if (x0 >= width) return;
    for (int y = (int)(blockIdx.y * 4 + (threadIdx.x >> 6)); y < height; y += (int)gridDim.y * 4) {
        const float* const in = src + (size_t)y * src_pitch;
        const size_t o = (size_t)y * dst_pitch;
        auto put = [&](int x, float v) {
            if constexpr (DTYPE == 1) ((_Float16*)dst)[o + x] = stored_f16(v, scale);
            else ((uint8_t*)dst)[o + x] = stored_u8(v, scale);
        };
        if constexpr (!VEC) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = in[min(x0 + kWaveSize * k, width - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (x0 + kWaveSize * k < width) put(x0 + kWaveSize * k, v[k]);
        } else if (x0 + 8 <= width) {
            const float4 a = *(const float4*)(in + x0), b = *(const float4*)(in + x0 + 4);
            const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            if constexpr (DTYPE == 1) {
                typedef _Float16 half8 __attribute__((ext_vector_type(8)));
                half8 h;
#pragma unroll
                for (int k = 0; k < 8; ++k) h[k] = stored_f16(v[k], scale);
                *(half8*)((_Float16*)dst + o + x0) = h;
            } else {
                unsigned w[2] = {0u, 0u};
#pragma unroll
                for (int k = 0; k < 8; ++k) w[k / 4] |= (unsigned)stored_u8(v[k], scale) << (8 * (k % 4));
                *(uint2*)((uint8_t*)dst + o + x0) = make_uint2(w[0], w[1]);
            }
        } else {
            for (int x = x0; x < width; ++x) put(x, in[x]);
        }
    }
}

// ---------------------------------------------------------- static scratch --
//
// Scratch of the allocation-free entry point (sgn_transfer_surfels_static): a
// file-scope device array, one copy per GPU, held until the process ends.
// Host code never uses the name `scratch` as an address: static_scratch_on
// looks up each device's copy once, with that device current, and the
// callers pass the looked-up pointer to kernels.
static __device__ __align__(256) unsigned char scratch[SGN_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch_on(int device, void** out) {
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return hipSuccess;
}

// ---------------------------------------------------------------- launchers --

hipError_t launch_stage(const void* host, void* dev, int n16, const FrameIn* in, FrameDev* frames, int n_frames,
                        uint32_t* counters, hipStream_t s) {
    const int blocks = (n16 + 255) / 256 + (n_frames + 255) / 256;
    hipLaunchKernelGGL(stage_kernel, dim3(blocks), dim3(256), 0, s, (const uint4*)host, (uint4*)dev, n16, in,
                       frames, n_frames, counters);
    return hipGetLastError();
}

// Workgroups of four wavefronts (the kernels stride over any that are left).
static dim3 wave_grid(int waves) { return dim3(std::max(1, std::min(1 << 20, (waves + 3) / 4))); }

hipError_t launch_init(const LoneKf& one, const BatchHeader* hdr, int waves, hipStream_t s) {
    hipLaunchKernelGGL(init_kernel, wave_grid(waves), dim3(256), 0, s, one, hdr);
    return hipGetLastError();
}

hipError_t launch_render(const LoneKf& one, const BatchHeader* hdr, int waves, hipStream_t s) {
    hipLaunchKernelGGL(render_kernel, wave_grid(waves), dim3(256), 0, s, one, hdr);
    return hipGetLastError();
}

hipError_t launch_quantize(const float* src, int src_pitch, void* dst, int dst_pitch, int width,
                           int height, int dtype, float scale, hipStream_t s) {
    const dim3 grid((width + 511) / 512, std::min(65535, (height + 3) / 4));
    const int unit = dtype == 1 ? 2 : 1;                       // bytes of a stored value
    const bool vec = ((uintptr_t)src & 15u) == 0 && (src_pitch & 3) == 0 &&
                     ((uintptr_t)dst & (8u * unit - 1u)) == 0 && (dst_pitch & 7) == 0;
    auto* f = dtype == 1 ? (vec ? quantize_kernel<1, true> : quantize_kernel<1, false>)
                         : (vec ? quantize_kernel<2, true> : quantize_kernel<2, false>);
    hipLaunchKernelGGL(f, grid, dim3(256), 0, s, src, src_pitch, dst, dst_pitch, width, height, scale);
    return hipGetLastError();
}

template <typename T, int S, int TX, int TY, int K, bool R, bool P, int D = 0, int SPLIT = 1, bool DAMPED = true>
static void* gn_ptr() {
    return (void*)&gn_kernel<T, S, TX, TY, K, R, D, SPLIT, P, DAMPED>;
}

template <typename T, int S, int TX, int TY, bool R, bool P, int KMAX = 4>
static void* gn_pick_groups(int groups) {
    if (groups == 1) return gn_ptr<T, S, TX, TY, 1, R, P>();
    if (groups == 2) return gn_ptr<T, S, TX, TY, 2, R, P>();
    if constexpr (KMAX >= 4)
        if (groups == 4) return gn_ptr<T, S, TX, TY, 4, R, P>();
    return nullptr;
}

template <typename T, bool R, bool P>
static void* gn_pick(const GnVariant& v) {
    if (v.patch == 8 && v.tiles_x == 1 && v.tiles_y == 1) return gn_pick_groups<T, 8, 1, 1, R, P>(v.groups);
    // a 16 x 16 surfel is its own anchor block: one group per item
    if (v.patch == 16 && v.tiles_x == 1 && v.tiles_y == 1 && v.groups == 1) return gn_ptr<T, 16, 1, 1, 1, R, P>();
    if (v.patch == 4 && v.tiles_x == 4 && v.tiles_y == 1) return gn_pick_groups<T, 4, 4, 1, R, P>(v.groups);
    if (v.patch == 4 && v.tiles_x == 2 && v.tiles_y == 2) return gn_pick_groups<T, 4, 2, 2, R, P>(v.groups);
    if (v.patch == 4 && v.tiles_x == 1 && v.tiles_y == 4) return gn_pick_groups<T, 4, 1, 4, R, P>(v.groups);
    // eight 4 x 4 surfels per wavefront, two pixels per lane: one or two groups
    if (v.patch == 4 && v.tiles_x == 4 && v.tiles_y == 2) return gn_pick_groups<T, 4, 4, 2, R, P, 2>(v.groups);
    if (v.patch == 4 && v.tiles_x == 2 && v.tiles_y == 4) return gn_pick_groups<T, 4, 2, 4, R, P, 2>(v.groups);
    // sixteen 4 x 4 surfels (a whole anchor block) per wavefront, four pixels per lane
    if (v.patch == 4 && v.tiles_x == 4 && v.tiles_y == 4 && v.groups == 1) return gn_ptr<T, 4, 4, 4, 1, R, P>();
    return nullptr;
}

// the forms for grids that leave the chip short of wavefronts (four pixels
// per lane: the 4x4 layout of 4x4 surfels, and 16 x 16 surfels)
template <typename T, bool R>
static void* gn_pick_deep(const GnVariant& v) {
    if (v.split == 4)
        return v.damped ? gn_ptr<T, 4, 2, 2, 1, R, false, 4, 4, true>() : gn_ptr<T, 4, 2, 2, 1, R, false, 4, 4, false>();
    if (v.split == 2)
        return v.damped ? gn_ptr<T, 4, 4, 2, 1, R, false, 2, 2, true>() : gn_ptr<T, 4, 4, 2, 1, R, false, 2, 2, false>();
    if (v.patch == 16) return v.deep == 2 ? gn_ptr<T, 16, 1, 1, 1, R, false, 2>() : gn_ptr<T, 16, 1, 1, 1, R, false, 1>();
    return v.deep == 2 ? gn_ptr<T, 4, 4, 4, 1, R, false, 2>() : gn_ptr<T, 4, 4, 4, 1, R, false, 1>();
}

// the form for large grids (f32 always has a frame's taps in flight)
template <typename T, bool R>
static void* gn_pick_shared(const GnVariant& v) {
    if constexpr (!std::is_same<T, float>::value)
        if (!v.deep)
            return v.patch == 16 ? (void*)&gn_shared_kernel<T, 16, 1, 1, R, 0> : (void*)&gn_shared_kernel<T, 4, 4, 4, R, 0>;
    return v.patch == 16 ? (void*)&gn_shared_kernel<T, 16, 1, 1, R, 1> : (void*)&gn_shared_kernel<T, 4, 4, 4, R, 1>;
}

template <typename T, bool R>
static void* gn_pick_form(const GnVariant& v) {
    if (v.shared) return gn_pick_shared<T, R>(v);
    return v.deep ? gn_pick_deep<T, R>(v) : gn_pick<T, R, false>(v);
}

template <typename T>
static void* gn_pick_rows(const GnVariant& v) {
    if (v.persistent) return v.by_row ? gn_pick<T, true, true>(v) : gn_pick<T, false, true>(v);
    return v.by_row ? gn_pick_form<T, true>(v) : gn_pick_form<T, false>(v);
}

static void* gn_select(const GnVariant& v) {
    if (v.lds) return nullptr;
    if (v.dtype == 0) return gn_pick_rows<float>(v);
    if (v.dtype == 1) return gn_pick_rows<_Float16>(v);
    if (v.dtype == 2) return gn_pick_rows<uint8_t>(v);
    return nullptr;
}

bool gn_variant_supported(const GnVariant& v) { return gn_select(v) != nullptr; }

// A kernel between the two timing events.  Recorded events: the launch that
// carries its own (hipExtLaunchKernel) took 6-7 us longer alone.
static hipError_t launch_timed(void* f, int grid_blocks, int threads, void** args, hipStream_t s, hipEvent_t start,
                               hipEvent_t stop, size_t lds = 0) {
    hipError_t e = hipEventRecord(start, s);
    if (e == hipSuccess) e = hipLaunchKernel(f, dim3(grid_blocks), dim3(threads), args, lds, s);
    if (e == hipSuccess) e = hipEventRecord(stop, s);
    return e;
}

hipError_t launch_gn(const GnVariant& v, const LoneBatch& one, const BatchHeader* hdr, uint32_t* counters,
                     int grid_blocks, hipStream_t s, hipEvent_t start, hipEvent_t stop) {
    void* f = gn_select(v);
    if (!f) return hipErrorInvalidValue;
    void* args[] = {(void*)&one, (void*)&hdr, (void*)&counters};      // (a shared kernel takes the first two)
    return launch_timed(f, grid_blocks, kBlockThreads, args, s, start, stop);
}

// ------------------------------------------------------------ disc surfels --
//
// Disc surfels (Eq. 4): surfel s is centred at u_s = (ux, uy) in keyframe
// pixels and covers the pixels u (inside the image) with |u - u_s| < r, r
// the same for every surfel of a keyframe (0 < r <= kDiscMaxRadius).
// Membership is decided as dx^2 + dy^2 < r^2 in double (dx = x - ux is
// exact there).  A disc's pixels are numbered row by row; a surfel held by
// LANES lanes gives lane l pixels l, l + LANES, ... (at most 512 / LANES).

constexpr int kDiscMaxRows = 2 * (int)kDiscMaxRadius + 2;
constexpr int kDiscPPL = 8;        // 512 pixels > pi (12 + sqrt(2)/2)^2, the largest disc
constexpr int kDiscRowWords = 2 * kDiscMaxRows + 2;
// largest ceil(beta r) of the neighbour search (beta <= 4, r <= 12)
constexpr int kDiscMaxWindowReach = 4 * (int)kDiscMaxRadius;

struct DiscRows {
    int y0, nrows, total;
};

// A disc pixel's slot in LDS: its offset from the anchor pixel as two int8
// (|offset| <= 12) in the low half-word and, for f16 and u8 images, the
// keyframe value's stored bits in the high half-word (f32 values go to a
// float array of their own).
template <typename T> struct DiscSlot {
    static constexpr bool packed = true;
};
template <> struct DiscSlot<float> {
    static constexpr bool packed = false;
};
__device__ __forceinline__ uint32_t slot_bits(_Float16 v) { return __builtin_bit_cast(uint16_t, v); }
__device__ __forceinline__ uint32_t slot_bits(uint8_t v) { return v; }
__device__ __forceinline__ uint32_t slot_bits(float) { return 0u; }
template <typename T>
__device__ __forceinline__ float slot_value(uint32_t pk);
template <>
__device__ __forceinline__ float slot_value<_Float16>(uint32_t pk) {
    return (float)__builtin_bit_cast(_Float16, (uint16_t)(pk >> 16));
}
template <>
__device__ __forceinline__ float slot_value<uint8_t>(uint32_t pk) { return (float)(pk >> 16); }
template <>
__device__ __forceinline__ float slot_value<float>(uint32_t) { return 0.f; }

// The rows of one disc (clipped to the image): the surfel's lanes below the
// row count (hl is the lane's index among the surfel's LANES lanes) find
// their row's run of pixels (a disc meets a row in one run), and a scan over
// those lanes forms the running counts.  row_x0[i] is the first column of
// row y0 + i and row_start[i] the number of disc pixels before it.  A
// non-finite centre gives an empty disc.  Every lane passes the same
// synchronisation point; the caller synchronises the wavefront before.
template <int LANES>
__device__ DiscRows disc_rows(float ux, float uy, float radius, int W, int H, int hl, int* row_x0,
                              int* row_start) {
#pragma clang fp contract(off)
    DiscRows d{0, 0, 0};
    const double cx = (double)ux, cy = (double)uy, r = (double)radius, r2 = r * r;
    const double xlo = fmax(0.0, ceil(cx - r)), xhi = fmin((double)(W - 1), floor(cx + r));
    const double ylo = fmax(0.0, ceil(cy - r)), yhi = fmin((double)(H - 1), floor(cy + r));
    const bool ok = isfinite(cx) && isfinite(cy) && xlo <= xhi && ylo <= yhi &&
                    yhi - ylo < (double)(kDiscMaxRows - 1);
    int x0 = 0, x1 = -1;
    if (ok) {
        x0 = (int)xlo;
        x1 = (int)xhi;
        d.y0 = (int)ylo;
        d.nrows = (int)yhi - d.y0 + 1;
    }
    int first = x0, cnt = 0;
    if (hl < d.nrows) {
        const double dy = (double)(d.y0 + hl) - cy;
        for (int x = x0; x <= x1; ++x) {
            const double dx = (double)x - cx;
            if (dx * dx + dy * dy < r2) {
                if (cnt == 0) first = x;
                ++cnt;
            }
        }
    }
    // inclusive scan of the row counts over the surfel's lanes
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1) {
        const int v = __shfl_up(incl, o, LANES);
        if (hl >= o) incl += v;
    }
    if (hl < d.nrows) {
        row_x0[hl] = first;
        row_start[hl + 1] = incl;
    }
    if (hl == 0) row_start[0] = 0;
    wave_sync();
    d.total = min(row_start[d.nrows], kWaveSize * kDiscPPL);
    return d;
}

// Pixel k (< total) of a disc.
__device__ __forceinline__ void disc_pixel(const DiscRows& d, const int* row_x0, const int* row_start,
                                           int k, int& x, int& y) {
    int i = 0;
    while (row_start[i + 1] <= k) ++i;
    x = row_x0[i] + (k - row_start[i]);
    y = d.y0 + i;
}

// Gauss-Newton over disc surfels: SPW surfels per wavefront, LANES = 64 /
// SPW lanes each (the batch's items are runs of SPW surfels of one keyframe),
// with the same per-pixel terms, frame loop, reduction and owner-lane step as
// the tile kernel, over the discs' pixels.  Each surfel's warp constants are
// anchored at the pixel nearest its centre.  With two surfels per wavefront
// the owner step (one lane per surfel) serves two surfels at once and the
// reductions span 32 lanes.  Six wavefronts per SIMD (80 VGPRs, and the LDS
// of six workgroups per CU): the few values that spill are read by the owner
// step once per iteration or by its double-precision fallback only.
//
// WAVES > 1: a workgroup of that many wavefronts per item, dealing out the
// pixel slots; each slot's A, B and cost go through LDS and every sum then runs
// over the slots in order, a pair of sums per wavefront, so the results are
// those of one wavefront.  DEEP as in frame_loop_px.  A lone wavefront takes
// about 22 us per iteration over a disc of radius 10 and six frames whatever
// the chip has free (640x480, 1,510 discs in 755 wavefronts: 324 us for 15
// iterations); four of them take 142 us, with the taps of four frames in
// flight.
//
// SHARED (undamped, an item per wavefront): one wavefront of the workgroup
// steps all its surfels, a lane each, as in gn_shared_kernel: the step is
// about 230 of the 4,400 VALU instructions that a wavefront issues per
// iteration over a disc of radius 10 and seven frames.  With the state in LDS
// and no damped branch, two frames in flight fit six wavefronts per SIMD where
// they held five; the pixels' and pair words' LDS is what the batch's largest
// disc and frame count need (22 KB where the most took 25).  VALU issue bounds
// it.  640x480, six frames: 511 -> 465 us at 9,060 discs (f16), 1,088 -> 982
// at 24,160; f32 607 -> 512 at 12,080 and 2,001 -> 1,810 at 48,320.  (One
// sample at a time at eight wavefronts: 481, 1,006; 533, 1,815.)
constexpr int disc_threads(int waves) { return waves == 1 ? kBlockThreads : waves * kWaveSize; }
template <int WAVES, int DEEP, bool SHARED>
constexpr int disc_waves() { return WAVES > 1 ? 4 : DEEP == 4 ? 4 : DEEP && !SHARED ? 5 : 6; }

template <typename T, int SPW, bool BY_ROW, int WAVES, int DEEP, bool SHARED>
__global__ __launch_bounds__(disc_threads(WAVES)) __attribute__((amdgpu_waves_per_eu(disc_waves<WAVES, DEEP, SHARED>(), 8))) void disc_gn_kernel(
    LoneBatch, const BatchHeader* __restrict__ hdr_, int total, int max_slots, int max_nbr) {
    constexpr int LANES = kWaveSize / SPW;        // lanes per surfel
    constexpr int PPL = kDiscPPL * SPW;           // pixel slots per lane
    constexpr int NWAVE = disc_threads(WAVES) / kWaveSize;
    constexpr int WPB = NWAVE / WAVES;            // items per workgroup
    static_assert(WAVES == 1 || WAVES == NWAVE, "an item takes a wavefront or a workgroup");
    constexpr bool packed = DiscSlot<T>::packed;
    static_assert(kDiscMaxRows <= LANES, "a disc row per lane");
    const BatchView view = batch_view(hdr_);
    const cptr<BatchHeader> hdr = view.hdr;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave_ = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wave = WAVES == 1 ? wave_ : 0;             // item of the workgroup
    const int part = WAVES == 1 ? 0 : wave_;             // wavefront of the item
    auto sync = [] {
        if constexpr (WAVES == 1) wave_sync();
        else __syncthreads();
    };
    const int h = lane / LANES, hl = lane % LANES;       // surfel of the wave, lane within it
    int first = (int)blockIdx.x * WPB, end = total;
    if (hdr->n_queues == kXcds) {
        // one share of the items per XCD (workgroups go to the XCDs in turn)
        const int share = (int)(blockIdx.x % (unsigned)kXcds);
        first = hdr->queues[share].begin + (int)(blockIdx.x / (unsigned)kXcds) * WPB;
        end = hdr->queues[share].end;
    }
    const int item = __builtin_amdgcn_readfirstlane(first + wave);
    const bool work = item < end;
    if (SHARED ? first >= end : !work) return;
    // (the shared form's pixels and pair words: as many as the batch needs)
    extern __shared__ float4 s_dyn[];
    __shared__ float4 s_pairs[SHARED ? 1 : WPB][SPW][kMaxNbr * kPairWords / 4];
    __shared__ float4 s_state[WPB][SPW][ST_WORDS / 4];
    __shared__ float4 s_sums[WPB][SPW][SM_WORDS / 4];
    __shared__ int s_rows[NWAVE][SPW][kDiscRowWords];
    // each lane's pixels: offsets from the anchor and keyframe values
    __shared__ uint32_t s_pix[SHARED ? 1 : WPB][PPL][kWaveSize];
    __shared__ float s_val[SHARED ? 1 : WPB][packed ? 1 : PPL][kWaveSize];
    // each slot's sums over the frames, and each wavefront's valid counts
    __shared__ float2 s_ab[WAVES > 1 ? PPL : 1][WAVES > 1 ? kWaveSize : 1];
    __shared__ float s_cst[WAVES > 1 ? PPL : 1][WAVES > 1 ? kWaveSize : 1];
    __shared__ int s_nv[WAVES > 1 ? NWAVE : 1][WAVES > 1 ? kWaveSize : 1];
    float* pairs;
    uint32_t (*pix)[kWaveSize];
    float (*vals)[kWaveSize];
    if constexpr (SHARED) {
        pairs = (float*)s_dyn + (wave * SPW + h) * max_nbr * kPairWords;
        uint32_t* const px = (uint32_t*)s_dyn + WPB * SPW * max_nbr * kPairWords;
        pix = (uint32_t (*)[kWaveSize])(px + wave * max_slots * kWaveSize);
        vals = (float (*)[kWaveSize])((float*)px + (WPB + wave) * max_slots * kWaveSize);
    } else {
        pairs = (float*)s_pairs[wave][h];
        pix = s_pix[wave];
        vals = s_val[wave];
    }
    float* const lst = (float*)s_state[wave][h];
    float* const lsm = (float*)s_sums[wave][h];
    int* const row_x0 = s_rows[wave_][h];
    int* const row_start = s_rows[wave_][h] + kDiscMaxRows;

    const cptr<KfDev> kfs = view.kfs;
    // a shared workgroup's wavefront without an item has no surfel and keeps to
    // the barriers
    const int kidx = !SHARED || work ? find_kf(kfs, hdr->n_kf, item, 0) : 0;
    const cptr<KfDev> Kd = kfs + kidx;
    const int sidx = (item - Kd->item_base) * SPW + h;
    const bool have = work && sidx < Kd->disc_count; // an odd count leaves the last half empty
    const int iters = hdr->iters;
    const float hk = hdr->huber_k;
    const float kap2 = hdr->kappa_fp64 * hdr->kappa_fp64;
    const bool depth_only = hdr->depth_only != 0;
    const float lm0 = hdr->lm_lambda;
    const bool lm = !SHARED && lm0 > 0.f;
    const int W = Kd->width, H = Kd->height;
    const int nf = Kd->n_nbr;
    const float img_scale = Kd->img_scale;
    const unsigned pitch_b = (unsigned)Kd->nbr_pitch_b;
    const unsigned wm1 = (unsigned)(W - 1), hm1 = (unsigned)(H - 1);
    const float fxk = Kd->fx, fyk = Kd->fy, cxk = Kd->cx, cyk = Kd->cy;
    const float ux = have ? ((gptr<float>)Kd->disc_ux)[sidx] : __builtin_nanf("");
    const float uy = have ? ((gptr<float>)Kd->disc_uy)[sidx] : __builtin_nanf("");

    wave_sync();                                     // (rows: each wavefront its own)
    const DiscRows d = disc_rows<LANES>(ux, uy, Kd->disc_r, W, H, hl, row_x0, row_start);
    // slot count: the larger of the wavefront's surfels, so the loop is uniform
    int nslots = (d.total + LANES - 1) / LANES;
    if constexpr (SPW == 2) nslots = max(nslots, __shfl_xor(nslots, 32));
    nslots = __builtin_amdgcn_readfirstlane(SHARED ? min(nslots, max_slots) : nslots);
    // anchor pixel (nearest the centre; any fixed point works for the local
    // warp coordinates)
    const int ax = (int)rint(fmin(fmax((double)ux, -1e6), 1e6));
    const int ay = (int)rint(fmin(fmax((double)uy, -1e6), 1e6));
    if (part == 0) stage_pair_words(view.frames + Kd->frame_base, nf, hl, (double)ax, (double)ay, pairs);
    const uint64_t fr_bits = (uint64_t)(view.frames + Kd->frame_base);
    const uint32_t fr_lo = __builtin_amdgcn_readfirstlane((uint32_t)fr_bits);
    const uint32_t fr_hi = __builtin_amdgcn_readfirstlane((uint32_t)(fr_bits >> 32));
    const cptr<FrameDev> fr = (cptr<FrameDev>)(((uint64_t)fr_hi << 32) | fr_lo);

    // this lane's pixels k = hl + LANES j, kept in LDS so that the slot loop
    // holds one pixel's terms in registers at a time
    const gptr<T> kimg = (gptr<T>)Kd->kf_img;
    const float kf_scale = Kd->kf_scale;
    for (int j = part; j < nslots; j += WAVES) {
        const int k = hl + LANES * j;
        uint32_t pk = 0u;
        float v = 0.f;
        if (k < d.total) {
            int x, y;
            disc_pixel(d, row_x0, row_start, k, x, y);
            const T raw = kimg[(unsigned)y * (unsigned)Kd->kf_pitch + (unsigned)x];
            pk = ((uint32_t)(x - ax) & 0xffu) | (((uint32_t)(y - ay) & 0xffu) << 8) | (slot_bits(raw) << 16);
            v = (float)raw * kf_scale;
        }
        pix[j][lane] = pk;
        if constexpr (!packed) vals[j][lane] = v;
    }
    // r_u - r_s = (anchor offset + (anchor - u_s)) / f
    const float fox = (float)((double)ax - (double)ux), foy = (float)((double)ay - (double)uy);
    const float ifx = 1.f / fxk, ify = 1.f / fyk;

    // owner (lane 0 of each surfel): the surfel's state
    const bool owner = hl == 0 && part == 0;
    const float rsx = (ux - cxk) / fxk, rsy = (uy - cyk) / fyk;
    float id = 0.f, nx = 0.f, ny = 0.f, nz = -1.f;
    uint32_t flags = 0u;
    if (have) {
        id = ((gptr<float>)Kd->inv_depth)[sidx];
        nx = ((gptr<float>)Kd->nx)[sidx];
        ny = ((gptr<float>)Kd->ny)[sidx];
        nz = ((gptr<float>)Kd->nz)[sidx];
        flags = ((gptr<uint32_t>)Kd->flags)[sidx] & ~F_GN_BITS;
    }
    bool alive = have, updated = false;
    float cost_out = 0.f;
    int nv_out = 0;
    float lam = lm0;
    float b1x = 0.f, b1y = 0.f, b1z = 0.f, b2x = 0.f, b2y = 0.f, b2z = 0.f;

    if constexpr (SHARED) {
        if (owner) {
            lst[ST_ID] = id; lst[ST_NX] = nx; lst[ST_NY] = ny; lst[ST_NZ] = nz;
            lst[ST_RSX] = rsx; lst[ST_RSY] = rsy;
            lst[ST_ALIVE] = have ? 1.f : 0.f;
            lst[ST_FLAGS] = __uint_as_float(flags);
            lst[ST_LAM] = 0.f;                       // set once a step is accepted
            lst[ST_COSTO] = 0.f; lst[ST_NVO] = __int_as_float(0);
            if (iters > 0) surfel_ready<true>(lst, nx, ny, nz, have, flags);
        }
    }

    for (int it = 0; it < iters; ++it) {
        const bool last = (it == iters - 1);
        if (!SHARED && owner) {
            const float c = nx * rsx + ny * rsy + nz;
            if (alive && fabsf(c) < 1e-6f) {
                flags |= F_DEGENERATE;
                alive = false;
                cost_out = 0.f;
                nv_out = 0;
            }
            tangent_basis(nx, ny, nz, b1x, b1y, b1z, b2x, b2y, b2z);
            lst[ST_ID] = id; lst[ST_NX] = nx; lst[ST_NY] = ny; lst[ST_NZ] = nz;
            lst[ST_B1X] = b1x; lst[ST_B1Y] = b1y; lst[ST_B1Z] = b1z;
            lst[ST_B2X] = b2x; lst[ST_B2Y] = b2y; lst[ST_B2Z] = b2z;
            lst[ST_INVC] = rcp_fast(c);
            lst[ST_RSX] = rsx; lst[ST_RSY] = rsy;
            lst[ST_ALIVE] = alive ? 1.f : 0.f;
        }
        if constexpr (SHARED) wave_sync();
        else sync();
        {
            const float4 sa = *(const float4*)(lst + 0);
            const float4 sb = *(const float4*)(lst + 4);
            const float4 sc = *(const float4*)(lst + 8);
            const float2 sd = *(const float2*)(lst + 12);
            const float sid = sa.x, snx = sa.y, sny = sa.z;
            const float sb1x = sb.x, sb1y = sb.y, sb1z = sb.z;
            const float sb2x = sb.w, sb2y = sc.x, sb2z = sc.y, inv_c = sc.z, srsx = sc.w;
            const float srsy = sd.x;
            const bool salive = sd.y != 0.f;
            // the surfel's parts of sigma_u and g_u (see gn_kernel), formed
            // once per iteration; the depth-only ablation zeroes kk
            const float cnx = snx * inv_c, cny = sny * inv_c;
            const float kk = depth_only ? 0.f : sid * inv_c;
            const float k1x = kk * sb1x, k1y = kk * sb1y, k2x = kk * sb2x, k2y = kk * sb2y;
            const float q1 = kk * fmaf(sb1x, srsx, fmaf(sb1y, srsy, sb1z));
            const float q2 = kk * fmaf(sb2x, srsx, fmaf(sb2y, srsy, sb2z));
            float ph[9] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            float pnv = 0.f, pcs = 0.f;
            const bool with_cost = last || lm;
            // one slot's pixel: offsets from the anchor, sigma_u and g_u
            struct Pixel {
                float bdx, bdy, sigma, g0, g1, g2;
            };
            auto pixel = [&](uint32_t pk) {
                Pixel x;
                x.bdx = (float)(int8_t)(pk & 0xffu);
                x.bdy = (float)(int8_t)((pk >> 8) & 0xffu);
                const float drx = (x.bdx + fox) * ifx, dry = (x.bdy + foy) * ify;
                x.sigma = fmaf(cny, dry, cnx * drx);
                x.g0 = 1.f + x.sigma;
                x.g1 = fmaf(-x.sigma, q1, fmaf(k1y, dry, k1x * drx));
                x.g2 = fmaf(-x.sigma, q2, fmaf(k2y, dry, k2x * drx));
                return x;
            };
            for (int j = part; j < nslots; j += WAVES) {
                const uint32_t pk = pix[j][lane];
                const Pixel x = pixel(pk);
                const float ikf[1] = {packed ? slot_value<T>(pk) * kf_scale : vals[packed ? 0 : j][lane]};
                const bool pv = hl + LANES * j < d.total;
                const float idu = fmaf(sid, x.sigma, sid);
                const bool pix_ok[1] = {salive && pv && (idu > 0.f)};
                float A[1] = {0.f}, B[1] = {0.f}, cst[1] = {0.f};
                unsigned nvl = 0u;
                if (with_cost)
                    frame_loop_px<T, true, 1, BY_ROW, DEEP, 1>(pairs, fr, nf, x.bdx, x.bdy, 0.f, idu, 0.f, 0, pix_ok,
                                                               pitch_b, wm1, hm1, ikf, hk, img_scale, A, B, cst, nvl);
                else
                    frame_loop_px<T, false, 1, BY_ROW, DEEP, 1>(pairs, fr, nf, x.bdx, x.bdy, 0.f, idu, 0.f, 0, pix_ok,
                                                                pitch_b, wm1, hm1, ikf, hk, img_scale, A, B, cst, nvl);
                pnv += (float)nvl;
                if constexpr (WAVES == 1) {
                    const float ag0 = A[0] * x.g0, ag1 = A[0] * x.g1, ag2 = A[0] * x.g2;
                    ph[0] = fmaf(ag0, x.g0, ph[0]); ph[1] = fmaf(ag0, x.g1, ph[1]);
                    ph[2] = fmaf(ag0, x.g2, ph[2]); ph[3] = fmaf(ag1, x.g1, ph[3]);
                    ph[4] = fmaf(ag1, x.g2, ph[4]); ph[5] = fmaf(ag2, x.g2, ph[5]);
                    ph[6] = fmaf(B[0], x.g0, ph[6]); ph[7] = fmaf(B[0], x.g1, ph[7]); ph[8] = fmaf(B[0], x.g2, ph[8]);
                    pcs += cst[0];
                } else {
                    s_ab[j][lane] = make_float2(A[0], B[0]);
                    if (with_cost) s_cst[j][lane] = cst[0];
                }
            }
            const bool odd = (hl & 1) != 0;
            if constexpr (WAVES == 1) {
#pragma clang fp contract(off)
                const float s0 = pair_sum<LANES>(ph[0], ph[1], odd);
                const float s1 = pair_sum<LANES>(ph[2], ph[3], odd);
                const float s2 = pair_sum<LANES>(ph[4], ph[5], odd);
                const float s3 = pair_sum<LANES>(ph[6], ph[7], odd);
                const float s4 = pair_sum<LANES>(ph[8], pnv, odd);
                float cs = 0.f;
                if (with_cost) cs = group_sum<LANES>(pcs);
                if (hl < 2) {
                    float* o = lsm + hl;
                    o[0] = s0; o[2] = s1; o[4] = s2; o[6] = s3; o[8] = s4;
                    if (hl == 0) o[SM_COST] = cs;
                }
            } else {
                s_nv[part][lane] = (int)pnv;
                sync();
                // wavefront p takes sums 2p and 2p + 1 (H00 H01, H02 H11, H12 H22,
                // b0 b1); the first also b2 and the count, the last the cost
                float e0 = 0.f, e1 = 0.f, e2 = 0.f;
                for (int j = 0; j < (part < 4 ? nslots : 0); ++j) {
                    const Pixel x = pixel(pix[j][lane]);
                    const float2 ab = s_ab[j][lane];
                    // the pair's factors: u0 v0 and u1 v1, u a product A g or B
                    const float ga = part < 2 ? x.g0 : part == 2 ? x.g1 : x.g0;
                    const float u0 = part == 3 ? ab.y : ab.x * ga;
                    const float v0 = part == 0 ? x.g0 : part == 3 ? x.g0 : x.g2;
                    const float u1 = part == 0 ? ab.x * x.g0 : part == 1 ? ab.x * x.g1
                                     : part == 2 ? ab.x * x.g2 : ab.y;
                    const float v1 = part == 2 ? x.g2 : x.g1;
                    e0 = fmaf(u0, v0, e0);
                    e1 = fmaf(u1, v1, e1);
                    if (part == 0) e2 = fmaf(ab.y, x.g2, e2);
                    if (part == 3 && with_cost) e2 += s_cst[j][lane];
                }
                const float se = pair_sum<LANES>(e0, e1, odd);
                if (hl < 2 && part < 4) lsm[2 * part + hl] = se;
                if (part == 0) {
                    int nvs = 0;
#pragma unroll
                    for (int w = 0; w < NWAVE; ++w) nvs += s_nv[w][lane];
                    const float s4 = pair_sum<LANES>(e2, (float)nvs, odd);
                    if (hl < 2) lsm[8 + hl] = s4;
                }
                if (part == 3) {
                    float cs = 0.f;
                    if (with_cost) cs = group_sum<LANES>(e2);
                    if (hl == 0) lsm[SM_COST] = cs;
                }
            }
        }
        if constexpr (SHARED) {
            __syncthreads();
            if (wave == (int)((blockIdx.x / kXcds + (unsigned)it) % WPB) && lane < WPB * SPW)
                shared_step<true>((float*)s_state + lane * ST_WORDS, (const float*)s_sums + lane * SM_WORDS, last,
                                  depth_only, kap2);
            __syncthreads();
            continue;
        }
        sync();
        bool cand = false;
        float id_c = 0.f, nx_c = 0.f, ny_c = 0.f, nz_c = 0.f, cost_here = 0.f;
        int nv = 0;
        if (owner)
            cand = owner_step(lsm, alive, last, depth_only, lm, kap2, lam, id, nx, ny, nz, b1x, b1y, b1z,
                              b2x, b2y, b2z, flags, cost_out, nv_out, nv, cost_here, id_c, nx_c, ny_c,
                              nz_c);
        if (WAVES == 1 && lm) {
            float inv_cc = 0.f;
            bool cand_ok = cand;
            if (owner && cand) {
                const float cc = nx_c * rsx + ny_c * rsy + nz_c;
                if (fabsf(cc) < 1e-6f) {             // candidate plane contains r_s
                    flags |= F_REJECTED;
                    lam *= 10.f;
                    cand_ok = false;
                }
                inv_cc = rcp_fast(cc);
            }
            if (owner) {
                lst[ST_ID] = id_c; lst[ST_NX] = nx_c; lst[ST_NY] = ny_c; lst[ST_NZ] = nz_c;
                lst[ST_INVC] = inv_cc;
                lst[ST_ALIVE] = cand_ok ? 1.f : 0.f;
            }
            wave_sync();
            {
                const float4 sa = *(const float4*)(lst + 0);
                const float inv_c = lst[ST_INVC];
                const bool calive = lst[ST_ALIVE] != 0.f;
                float cst2 = 0.f;
                int nv2l = 0;
                for (int j = 0; j < nslots; ++j) {
                    const uint32_t pk = pix[j][lane];
                    const float bdx = (float)(int8_t)(pk & 0xffu), bdy = (float)(int8_t)((pk >> 8) & 0xffu);
                    const float ikf = packed ? slot_value<T>(pk) * kf_scale : vals[packed ? 0 : j][lane];
                    const bool pv = hl + LANES * j < d.total;
                    const float drx = (bdx + fox) * ifx, dry = (bdy + foy) * ify;
                    const float sig = fmaf(sa.z * inv_c, dry, (sa.y * inv_c) * drx);
                    const float idu_c = fmaf(sa.x, sig, sa.x);
                    frame_cost<T, BY_ROW, DEEP>(pairs, fr, nf, bdx, bdy, idu_c, calive && pv && (idu_c > 0.f), pitch_b,
                                                wm1, hm1, ikf, hk, img_scale, cst2, nv2l);
                }
                const float c2 = group_sum<LANES>(cst2);
                const int n2 = group_sum<LANES>(nv2l);
                if (hl == 0) {
                    lsm[SM_COST] = c2;
                    lsm[SM_NV] = __int_as_float(n2);
                }
            }
            wave_sync();
            if (owner && cand_ok) cand_ok = lm_accept(lsm[SM_COST], __float_as_int(lsm[SM_NV]), cost_here, nv, lam);
            cand = cand_ok;
        }
        if (owner && cand) {
            id = id_c;
            nx = nx_c; ny = ny_c; nz = nz_c;
            updated = true;
        }
    }
    if constexpr (SHARED) {
        id = lst[ST_ID]; nx = lst[ST_NX]; ny = lst[ST_NY]; nz = lst[ST_NZ];
        flags = __float_as_uint(lst[ST_FLAGS]);
        cost_out = lst[ST_COSTO]; nv_out = __float_as_int(lst[ST_NVO]);
        updated = lst[ST_LAM] != 0.f;
    }
    if (owner && have) {
        ((gmut<float>)Kd->inv_depth)[sidx] = id;
        ((gmut<float>)Kd->nx)[sidx] = nx;
        ((gmut<float>)Kd->ny)[sidx] = ny;
        ((gmut<float>)Kd->nz)[sidx] = nz;
        ((gmut<uint32_t>)Kd->flags)[sidx] = flags;
        ((gmut<float>)Kd->cost)[sidx] = iters > 0 ? cost_out : 0.f;
        ((gmut<uint32_t>)Kd->nvalid)[sidx] = (uint32_t)(iters > 0 ? nv_out : 0);
        if (updated) ((gmut<uint32_t>)Kd->last_update)[sidx] = hdr->stamp;
    }
}

// Depth-buffered render (Inverse Depth Calculation section): every usable
// surfel (no DEGENERATE or UNINIT flag, finite centre, plane not through its
// centre ray) writes Eq. 3 into the pixels of its disc; the closest (largest
// id_u > 0) wins and equal values go to the lower index.  id_u is evaluated
// in double in the printed form of Eq. 3, id_u = (r_u . n) / ((r_s / id_s) . n).
//
// The render works in screen tiles of kRenderTile x kRenderTile pixels.  The
// usable surfels are binned to the tiles their disc's bounding box meets (a
// count per tile, a range of the list for each, a fill); then a wavefront or
// four per tile walk the tile's list keeping, for each pixel, the largest value
// and the lowest index that reaches it.  The outcome does not depend on the
// list order, so the fill's atomics leave it deterministic, and the depth test
// needs no atomics.
//
// Binning takes one launch, a workgroup per keyframe (disc_bin_lds_kernel,
// where bin_in_lds says so), else four over the whole device (clear, count,
// ranges, fill).  For few surfels the launches count, about 4.7 us each: a
// 640x480 keyframe's render took 35 us with seven (three of them a scan of
// the counts) and takes 17 with two.

// Table entry of global surfel g (largest surfel_base <= g among entries
// with surfels) or of global tile t (by tile_base).
__device__ __forceinline__ int render_item_of_surfel(cptr<DiscRenderItem> tab, int n, int g) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tab[mid].surfel_base <= g) lo = mid; else hi = mid - 1;
    }
    return lo;        // entries without surfels share the next base and are never the largest
}
__device__ __forceinline__ int render_item_of_tile(cptr<DiscRenderItem> tab, int n, int t) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tab[mid].tile_base <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

__global__ void fill_int_kernel(int32_t* __restrict__ p, int n, int32_t v) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = v;
}

// The tiles that surfel s's disc (its bounding box inside the image) meets.
struct TileBox {
    int tx0, tx1, ty0, ty1;
};
__device__ __forceinline__ bool disc_box(const carg<DiscRenderItem>& a, int s, TileBox& b) {
    const double cx = (double)a.ux[s], cy = (double)a.uy[s], r = (double)a.radius;
    if (!isfinite(cx) || !isfinite(cy)) return false;
    const double xlo = fmax(0.0, ceil(cx - r)), xhi = fmin((double)(a.width - 1), floor(cx + r));
    const double ylo = fmax(0.0, ceil(cy - r)), yhi = fmin((double)(a.height - 1), floor(cy + r));
    if (!(xlo <= xhi) || !(ylo <= yhi)) return false;
    b.tx0 = (int)xlo / kRenderTile; b.tx1 = (int)xhi / kRenderTile;
    b.ty0 = (int)ylo / kRenderTile; b.ty1 = (int)yhi / kRenderTile;
    return true;
}
// Whether surfel s is drawn, with its raster record and tiles.
__device__ __forceinline__ bool disc_record(const carg<DiscRenderItem>& a, int s, DiscRaster& rec, TileBox& b) {
#pragma clang fp contract(off)
    // every load before the first test (one round trip)
    const uint32_t fl = a.flags[s];
    const double cx = (double)a.ux[s], cy = (double)a.uy[s];
    const double n0 = a.nx[s], n1 = a.ny[s], n2 = a.nz[s], ids = a.inv_depth[s];
    if (fl & (F_DEGENERATE | F_UNINIT)) return false;
    if (!disc_box(a, s, b)) return false;
    const double rs0 = (cx - a.cx) / a.fx, rs1 = (cy - a.cy) / a.fy;
    if (fabs(n0 * rs0 + n1 * rs1 + n2 * 1.0) < 1e-6) return false;
    const double ps0 = rs0 / ids, ps1 = rs1 / ids, ps2 = 1.0 / ids;
    rec = DiscRaster{cx, cy, n0, n1, n2, ps0 * n0 + ps1 * n1 + ps2 * n2};
    return true;
}

__global__ __launch_bounds__(256) void disc_count_kernel(DiscRenderItem, const DiscRenderItem* __restrict__ tab_,
                                                         int n_items, int total, DiscRaster* __restrict__ rec,
                                                         int32_t* __restrict__ count) {
    const cptr<DiscRenderItem> tab = table_or_arg(tab_);
    const int g = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (g >= total) return;
    const carg<DiscRenderItem>& a = tab[render_item_of_surfel(tab, n_items, g)];
    DiscRaster q;
    TileBox b;
    const bool use = disc_record(a, g - a.surfel_base, q, b);
    if (!use) q.cx = __builtin_nan("");          // the fill skips it
    rec[g] = q;
    if (!use) return;
    for (int ty = b.ty0; ty <= b.ty1; ++ty)
        for (int tx = b.tx0; tx <= b.tx1; ++tx) atomicAdd(count + a.tile_base + ty * a.tiles_x + tx, 1);
}

__global__ __launch_bounds__(256) void disc_fill_kernel(DiscRenderItem, const DiscRenderItem* __restrict__ tab_,
                                                        int n_items, int total, const DiscRaster* __restrict__ rec,
                                                        int32_t* __restrict__ start, int32_t* __restrict__ list) {
    const cptr<DiscRenderItem> tab = table_or_arg(tab_);
    const int g = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (g >= total) return;
    const carg<DiscRenderItem>& a = tab[render_item_of_surfel(tab, n_items, g)];
    TileBox b;
    if (isnan(rec[g].cx) || !disc_box(a, g - a.surfel_base, b)) return;
    for (int ty = b.ty0; ty <= b.ty1; ++ty)
        for (int tx = b.tx0; tx <= b.tx1; ++tx)
            list[atomicSub(start + a.tile_base + ty * a.tiles_x + tx, 1) - 1] = g;
}

// Exclusive scan over a workgroup of up to 1024 threads; s_w holds 17 words.
__device__ __forceinline__ int block_exclusive_scan(int v, int* s_w, int& block_total) {
    const int lane = threadIdx.x & (kWaveSize - 1), wave = threadIdx.x >> 6;
    int x = v;
#pragma unroll
    for (int o = 1; o < kWaveSize; o <<= 1) {
        const int y = __shfl_up(x, o, kWaveSize);
        if (lane >= o) x += y;
    }
    if (lane == kWaveSize - 1) s_w[wave] = x;
    __syncthreads();
    if (wave == 0) {
        // the wavefronts' sums, one per lane (at most sixteen)
        const int n = (int)(blockDim.x / kWaveSize);
        const int c = lane < n ? s_w[lane] : 0;
        int w = c;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            const int y = __shfl_up(w, o, kWaveSize);
            if (lane >= o) w += y;
        }
        if (lane < n) s_w[lane] = w - c;
        if (lane == n - 1) s_w[16] = w;
    }
    __syncthreads();
    block_total = s_w[16];
    const int ex = s_w[wave] + x - v;
    __syncthreads();
    return ex;
}
// A range of the list for each tile, in no particular order: a scan within
// each workgroup and one atomic per workgroup on the list's cursor.  start[t]
// is the range's end; the fill counts it down to the beginning.
__global__ __launch_bounds__(1024) void disc_range_kernel(const int32_t* __restrict__ count,
                                                          int32_t* __restrict__ start, int32_t* __restrict__ cursor,
                                                          int n) {
    __shared__ int s_w[17];
    __shared__ int s_base;
    const int i = (int)(blockIdx.x * 1024 + threadIdx.x);
    const int c = i < n ? count[i] : 0;
    int tot;
    const int ex = block_exclusive_scan(c, s_w, tot);
    if (threadIdx.x == 0) s_base = atomicAdd(cursor, tot);
    __syncthreads();
    if (i < n) start[i] = s_base + ex + c;
}

// The whole binning of one keyframe in a workgroup, its tile counts in LDS.
// The keyframe's part of the list begins at its first surfel's entries.
__global__ __launch_bounds__(1024) void disc_bin_lds_kernel(DiscRenderItem, const DiscRenderItem* __restrict__ tab_,
                                                            DiscRaster* __restrict__ rec,
                                                            int32_t* __restrict__ count, int32_t* __restrict__ start,
                                                            int32_t* __restrict__ list) {
    const cptr<DiscRenderItem> tab = table_or_arg(tab_);
    const carg<DiscRenderItem>& a = tab[blockIdx.x];
    __shared__ int s_cnt[kBinTiles];
    __shared__ unsigned long long s_use[(kBinSurfels + kWaveSize - 1) / kWaveSize];
    __shared__ int s_w[17];
    const int tid = (int)threadIdx.x;
    const int tiles = a.tiles_x * ((a.height + kRenderTile - 1) / kRenderTile);
    for (int t = tid; t < tiles; t += 1024) s_cnt[t] = 0;
    __syncthreads();
    const int n64 = (a.count + kWaveSize - 1) & ~(kWaveSize - 1);       // whole wavefronts
    for (int s = tid; s < n64; s += 1024) {
        DiscRaster q;
        TileBox b;
        const bool use = s < a.count && disc_record(a, s, q, b);
        const unsigned long long ball = __ballot(use);
        if ((tid & (kWaveSize - 1)) == 0) s_use[s / kWaveSize] = ball;
        if (!use) continue;
        rec[a.surfel_base + s] = q;
        for (int ty = b.ty0; ty <= b.ty1; ++ty)
            for (int tx = b.tx0; tx <= b.tx1; ++tx) atomicAdd(&s_cnt[ty * a.tiles_x + tx], 1);
    }
    __syncthreads();
    // each thread takes a run of tiles: one scan over the workgroup
    const int run = (tiles + 1023) / 1024;
    const int t0 = min(tiles, tid * run), t1 = min(tiles, t0 + run);
    int sum = 0;
    for (int t = t0; t < t1; ++t) sum += s_cnt[t];
    int tot;
    int at = kDiscMaxTilesPerSurfel * a.surfel_base + block_exclusive_scan(sum, s_w, tot);
    for (int t = t0; t < t1; ++t) {
        const int c = s_cnt[t];
        s_cnt[t] = at;
        at += c;
    }
    __syncthreads();
    const int end = kDiscMaxTilesPerSurfel * a.surfel_base + tot;
    for (int t = tid; t < tiles; t += 1024) {
        start[a.tile_base + t] = s_cnt[t];
        count[a.tile_base + t] = (t + 1 < tiles ? s_cnt[t + 1] : end) - s_cnt[t];
    }
    __syncthreads();
    for (int s = tid; s < a.count; s += 1024) {
        TileBox b;
        if (!((s_use[s / kWaveSize] >> (s & (kWaveSize - 1))) & 1ull) || !disc_box(a, s, b)) continue;
        for (int ty = b.ty0; ty <= b.ty1; ++ty)
            for (int tx = b.tx0; tx <= b.tx1; ++tx)
                list[atomicAdd(&s_cnt[ty * a.tiles_x + tx], 1)] = a.surfel_base + s;
    }
}

// A wavefront per tile with four pixels of one column per lane (PX = 4), or
// four wavefronts with one (see raster_pixels): the largest Eq. 3 value over
// the tile's surfels whose disc holds the pixel, and the lowest index among
// those that reach it.  The tile's list is staged in LDS, 64 entries at a time
// (one entry and its raster record per lane, all loads in flight at once).
//
// Bound: the chain of dependent loads in front of the walk (keyframe, range,
// list, records), so what counts is how many tiles a CU holds: 32 with a
// wavefront each, where four-wavefront workgroups left eight.  Renders of 1 /
// 8 / 32 keyframes of 1280x720 with 4,641 discs: 37 / 84 / 246 us with a
// workgroup per tile, 29 / 63 / 159 now.  (Choosing by num * (1 / den), with
// divisions only where two products come near each other: 29 / 65 / 165, and
// 34 / 88 / 254 where all surfels lie on one plane.)
template <int PX>
__global__ __launch_bounds__(kBlockThreads) void disc_raster_kernel(
    DiscRenderItem, const DiscRenderItem* __restrict__ tab_, int n_items, int n_tiles,
    const DiscRaster* __restrict__ rec, const int32_t* __restrict__ count, const int32_t* __restrict__ start,
    const int32_t* __restrict__ list) {
#pragma clang fp contract(off)
    const cptr<DiscRenderItem> tab = table_or_arg(tab_);
    constexpr int kParts = kRenderTile * kRenderTile / (PX * kWaveSize);      // wavefronts per tile
    static_assert(kRenderTile == 16 && kParts * PX * kWaveSize == kRenderTile * kRenderTile, "tiles in whole wavefronts");
    __shared__ DiscRaster s_rec_[kBlockThreads / kWaveSize][kWaveSize];
    __shared__ int s_idx_[kBlockThreads / kWaveSize][kWaveSize];
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    DiscRaster* const s_rec = s_rec_[wave];
    int* const s_idx = s_idx_[wave];
    const int t = grid_wave() / kParts, part = grid_wave() % kParts;
    if (t >= n_tiles) return;
    const carg<DiscRenderItem>& a = tab[render_item_of_tile(tab, n_items, t)];
    const int lt = t - a.tile_base;
    const int ty = lt / a.tiles_x, tx = lt - ty * a.tiles_x;
    const int x = tx * kRenderTile + (lane & (kRenderTile - 1));
    const int y0 = ty * kRenderTile + 4 * PX * part + lane / kRenderTile;      // rows y0, y0 + 4, ...
    const double r = (double)a.radius, r2 = r * r;
    const double xd = (double)x, ru0 = (xd - a.cx) / a.fx;
    double yd[PX], ru1[PX], val[PX];
    int who[PX];
#pragma unroll
    for (int p = 0; p < PX; ++p) {
        yd[p] = (double)(y0 + 4 * p);
        ru1[p] = (yd[p] - a.cy) / a.fy;
        val[p] = 0.0;
        who[p] = -1;
    }
    const int k0 = start[t], k1 = k0 + count[t];
    for (int c0 = k0; c0 < k1; c0 += kWaveSize) {
        const int nc = min(kWaveSize, k1 - c0);
        wave_sync();                          // the previous chunk is read
        if (lane < nc) {
            const int g = list[c0 + lane];
            s_idx[lane] = g - a.surfel_base;
            s_rec[lane] = rec[g];
        }
        wave_sync();
        for (int e = 0; e < nc; ++e) {
            const DiscRaster q = s_rec[e];
            const int idx = s_idx[e];
            const double dx = xd - q.cx, dx2 = dx * dx;
            const double nx = ru0 * q.n0;
#pragma unroll
            for (int p = 0; p < PX; ++p) {
                const double dy = yd[p] - q.cy;
                // (a branch: most entries miss all of a row group's pixels)
                if (!(dx2 + dy * dy < r2)) continue;
                const double v = (nx + ru1[p] * q.n1 + 1.0 * q.n2) / q.den;
                if (!(v > 0.0) || !isfinite(v)) continue;
                if (v > val[p] || (v == val[p] && idx < who[p])) {
                    val[p] = v;
                    who[p] = idx;
                }
            }
        }
    }
#pragma unroll
    for (int p = 0; p < PX; ++p) {
        const int y = y0 + 4 * p;
        if (x >= a.width || y >= a.height) continue;
        const size_t o = (size_t)y * (size_t)a.width + (size_t)x;
        a.inv_depth_out[o] = (float)val[p];
        if (a.index_out) a.index_out[o] = who[p];
    }
}

// Placement runs over a table of keyframes (up to kDiscPlaceArgs of them in the
// kernels' arguments, as in the disc transfer): candidates and new surfels are
// numbered keyframe after keyframe (cand_base, init_base); the entry owning
// number g is the last whose base is <= g (entries with none share the next
// base and are never the last).
template <int N>
struct DiscPlaceTab {
    DiscPlaceArgs item[N];
};
__device__ __forceinline__ int place_entry_of_cand(cptr<DiscPlaceArgs> tab, int n, int g) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tab[mid].cand_base <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}
__device__ __forceinline__ int place_entry_of_init(cptr<DiscPlaceArgs> tab, int n, int g) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (tab[mid].init_base <= g) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Pixel k of the side x side window of pixels within `reach` of (cx, cy), its
// place in the index map clamped to the image, so that it can be loaded
// whether it lies inside or not (a load inside a branch is waited for there).
// k / side is a multiplication by inv = floor(2^20 / side) + 1, exact for
// k below 2^20 / side - side: the largest window has 97 x 97 pixels.
struct WindowPixel {
    int dx, dy, at;
    bool inside;
};
__device__ __forceinline__ unsigned window_inv(int side) { return (1u << 20) / (unsigned)side + 1u; }
__device__ __forceinline__ WindowPixel window_pixel(int k, int side, int reach, unsigned inv, int cx, int cy, int W,
                                                    int H) {
    const int row = (int)(((unsigned)k * inv) >> 20);
    WindowPixel w;
    w.dy = row - reach;
    w.dx = k - row * side - reach;
    const int x = cx + w.dx, y = cy + w.dy;
    w.inside = x >= 0 && y >= 0 && x < W && y < H;
    w.at = min(max(y, 0), H - 1) * W + min(max(x, 0), W - 1);
    return w;
}

// The search for empty areas (Surfel Initialization section): one wavefront
// per lattice candidate u_ns = (spacing/2 + i spacing, spacing/2 + j
// spacing), its lanes sharing the window of pixels within alpha r; the
// candidate qualifies when no non-empty pixel of the index map lies within
// alpha r (integer squared distance against (alpha r)^2 in double).
template <int N>
__global__ __launch_bounds__(kBlockThreads) void disc_search_kernel(DiscPlaceTab<N>, const DiscPlaceArgs* __restrict__ tab_,
                                                                    int n_items, int total) {
    const cptr<DiscPlaceArgs> tab = table_or_arg(tab_);
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int g = __builtin_amdgcn_readfirstlane((int)blockIdx.x * (kBlockThreads / kWaveSize) +
                                                 (int)(threadIdx.x >> 6));
    if (g >= total) return;
    const carg<DiscPlaceArgs>& a = tab[place_entry_of_cand(tab, n_items, g)];
    const int c = g - a.cand_base;
    const int cx = a.spacing / 2 + (c % a.cand_x) * a.spacing;
    const int cy = a.spacing / 2 + (c / a.cand_x) * a.spacing;
    const double ar = (double)a.alpha * (double)a.radius;
    const double ar2 = ar * ar;
    const int reach = (int)floor(ar);
    const int side = 2 * reach + 1, npix = side * side;
    const unsigned inv = window_inv(side);
    // Bound by the loads' latency, candidate by candidate.  The first 64 pixels
    // alone: on a map that is mostly full they decide nearly every candidate.
    // Then four pixels per lane in flight, only those inside the window.  A
    // placement, one pixel at a time / four from the start / so: full map
    // 1572x1230, 2 keyframes, spacing 2, 488 / 570 / 465 us; half empty 1476x1065,
    // 5 keyframes, radius 4.5 (81 pixels) 99 / 103 / 99, 1152x886, 7 keyframes,
    // radius 9.4 77 / 63 / 60.
    bool hit = false;
    if (lane < npix) {
        const WindowPixel w = window_pixel(lane, side, reach, inv, cx, cy, a.width, a.height);
        hit = w.inside && (double)(w.dx * w.dx + w.dy * w.dy) <= ar2 && a.index_map[w.at] >= 0;
    }
    for (int k0 = kWaveSize; k0 < npix; k0 += 4 * kWaveSize) {
        if (__ballot(hit) != 0ull) break;     // wave-uniform
        int own[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = k0 + u * kWaveSize + lane;
            const WindowPixel w = window_pixel(k, side, reach, inv, cx, cy, a.width, a.height);
            own[u] = -1;
            if (k < npix && w.inside && (double)(w.dx * w.dx + w.dy * w.dy) <= ar2) own[u] = a.index_map[w.at];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) hit = hit || own[u] >= 0;
    }
    // the vote of the whole wavefront, taken before narrowing to one lane
    const bool empty = __ballot(hit) == 0ull;
    if (lane == 0) a.cand_flag[c] = empty ? 1 : 0;
}

// Placement: the qualifying candidates in lattice order become surfels
// first, first + 1, ... (as many as there is room for); counts[0] = placed,
// counts[1] = qualifying.  One workgroup per keyframe scans its flags in
// chunks.
template <int N>
__global__ __launch_bounds__(1024) void disc_compact_kernel(DiscPlaceTab<N>, const DiscPlaceArgs* __restrict__ tab_) {
    const cptr<DiscPlaceArgs> tab = table_or_arg(tab_);
    const carg<DiscPlaceArgs>& a = tab[blockIdx.x];
    __shared__ int s_wave[1024 / kWaveSize + 1];
    const int n = a.cand_x * a.cand_y;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    constexpr int kWaves = 1024 / kWaveSize;
    int base = 0;
    for (int c0 = 0; c0 < n; c0 += 1024) {
        const int c = c0 + (int)threadIdx.x;
        const bool f = c < n && a.cand_flag[c] != 0;
        const unsigned long long ball = __ballot(f);
        const int below = __popcll(ball & ((1ull << lane) - 1ull));
        if (lane == 0) s_wave[wave] = __popcll(ball);
        __syncthreads();
        if (threadIdx.x == 0) {
            int acc = 0;
            for (int w = 0; w < kWaves; ++w) {
                const int t = s_wave[w];
                s_wave[w] = acc;
                acc += t;
            }
            s_wave[kWaves] = acc;
        }
        __syncthreads();
        const int rank = base + s_wave[wave] + below;
        if (f && rank < a.room) {
            const int cx = a.spacing / 2 + (c % a.cand_x) * a.spacing;
            const int cy = a.spacing / 2 + (c / a.cand_x) * a.spacing;
            a.ux[a.first + rank] = (float)cx;
            a.uy[a.first + rank] = (float)cy;
        }
        base += s_wave[kWaves];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.counts[0] = min(base, a.room);
        a.counts[1] = base;
    }
}

// The minimum over the wavefront, in every lane: within DPP rows of sixteen,
// then over the four rows through scalar registers.
__device__ __forceinline__ int wave_min(int v) {
    v = min(v, dpp_i<0xB1>(v));      // quad_perm [1,0,3,2]
    v = min(v, dpp_i<0x4E>(v));      // quad_perm [2,3,0,1]
    v = min(v, dpp_i<0x141>(v));     // row_half_mirror
    v = min(v, dpp_i<0x140>(v));     // row_mirror
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// Neighbour initialisation of the placed surfels (Surfel Initialization
// section), one wavefront each: the neighbours are the surfels below
// `first` that own a pixel of the index map closer than beta r to the new
// centre, visited in index order (the wavefront finds the next smallest
// index each round); id = mean of Eq. 3 of their planes at the new ray,
// n = mean of their normals sign-aligned to the first, renormalised; none
// usable: UNINIT with id 0 and n = (0, 0, -1).  The indices are found first,
// one lane each, and all their surfels loaded together, as are the window's
// pixels: bound by latency, a 640x480 keyframe's new surfels took 21 us with
// the loads one after another and take 11.  SLOTS pixels per lane: nine, or two
// where that covers every window, which a placement of many small discs pays
// for (4 empty 640x480 maps, radius 1.5: 672 us one at a time, 798 with nine,
// 577 with two).
template <int N, int SLOTS>
__global__ __launch_bounds__(kWaveSize) void disc_init_kernel(DiscPlaceTab<N>, const DiscPlaceArgs* __restrict__ tab_,
                                                              int n_items) {
    const cptr<DiscPlaceArgs> tab = table_or_arg(tab_);
    // the window's surfel indices (those within beta r, below `first`), or -1
    __shared__ int s_win[(2 * kDiscMaxWindowReach + 1) * (2 * kDiscMaxWindowReach + 1)];
    const int lane = threadIdx.x;
    const int g = __builtin_amdgcn_readfirstlane((int)blockIdx.x);
    const carg<DiscPlaceArgs>& a = tab[place_entry_of_init(tab, n_items, g)];
    const int w = g - a.init_base;
    if (w >= a.counts[0]) return;
    const int i = a.first + w;
    const int cx = (int)a.ux[i], cy = (int)a.uy[i];
    const double br = (double)a.beta * (double)a.radius;
    const double br2 = br * br;
    const int reach = (int)ceil(br);
    const int side = 2 * reach + 1, npix = side * side;
    const unsigned inv = window_inv(side);
    // SLOTS pixels per lane in flight at a time
    for (int k0 = 0; k0 < npix; k0 += SLOTS * kWaveSize) {
        int own[SLOTS];
        bool in[SLOTS];
#pragma unroll
        for (int u = 0; u < SLOTS; ++u) {
            const WindowPixel w = window_pixel(k0 + u * kWaveSize + lane, side, reach, inv, cx, cy, a.width, a.height);
            in[u] = w.inside && (double)(w.dx * w.dx + w.dy * w.dy) < br2;
            own[u] = a.index_map[w.at];
        }
#pragma unroll
        for (int u = 0; u < SLOTS; ++u) {
            const int k = k0 + u * kWaveSize + lane;
            if (k < npix) s_win[k] = in[u] && own[u] < a.first ? own[u] : -1;
        }
    }
    wave_sync();
    const float rnx = ((float)cx - a.cx) / a.fx, rny = ((float)cy - a.cy) / a.fy;
    int last = -1, count = 0;
    float id_sum = 0.f, sx = 0.f, sy = 0.f, sz = 0.f, rx = 0.f, ry = 0.f, rz = 0.f;
    for (bool more = true; more;) {
        // the next 64 neighbours in index order, one per lane
        int mine = -1, found = 0;
        while (found < kWaveSize) {
            int best = 0x7fffffff;
            for (int k = lane; k < npix; k += kWaveSize) {
                const int j = s_win[k];
                if (j > last) best = min(best, j);
            }
            best = wave_min(best);
            if (best == 0x7fffffff) {
                more = false;
                break;
            }
            last = best;
            if (lane == found) mine = best;
            ++found;
        }
        // every lane's neighbour at once: usable, its Eq. 3 at the new
        // surfel's ray, its normal
        bool use = mine >= 0;
        float id = 0.f, njx = 0.f, njy = 0.f, njz = 0.f;
        if (use) {
            const uint32_t fl = a.flags[mine];
            njx = a.nx[mine]; njy = a.ny[mine]; njz = a.nz[mine];
            const float ujx = a.ux[mine], ujy = a.uy[mine], idj = a.inv_depth[mine];
            const float rjx = (ujx - a.cx) / a.fx, rjy = (ujy - a.cy) / a.fy;
            const float cj = njx * rjx + njy * rjy + njz;
            use = !(fl & (F_UNINIT | F_DEGENERATE)) && !(fabsf(cj) < 1e-6f);
            id = idj * (njx * rnx + njy * rny + njz) / cj;
        }
        // summed in index order
        for (unsigned long long m = __ballot(use); m != 0ull; m &= m - 1ull) {
            const int l = __builtin_ctzll(m);
            auto of = [&](float v) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
            const float jx = of(njx), jy = of(njy), jz = of(njz);
            if (count == 0) { rx = jx; ry = jy; rz = jz; }
            const float sg = (jx * rx + jy * ry + jz * rz) < 0.f ? -1.f : 1.f;
            id_sum += of(id);
            sx += sg * jx; sy += sg * jy; sz += sg * jz;
            ++count;
        }
    }
    if (lane != 0) return;
    bool ok = count > 0;
    float idn = 0.f, l2 = 0.f;
    if (ok) {
        const float inv = 1.0f / (float)count;
        idn = id_sum * inv;
        sx *= inv; sy *= inv; sz *= inv;
        l2 = sx * sx + sy * sy + sz * sz;
        ok = (l2 > 0.f) && (idn > 0.f) && isfinite(idn) && isfinite(l2);
    }
    if (ok) {
        const float il = 1.0f / sqrtf(l2);
        a.inv_depth[i] = idn;
        a.nx[i] = sx * il; a.ny[i] = sy * il; a.nz[i] = sz * il;
        a.flags[i] = 0u;
    } else {
        a.inv_depth[i] = 0.f;
        a.nx[i] = 0.f; a.ny[i] = 0.f; a.nz[i] = -1.f;
        a.flags[i] = F_UNINIT;
    }
    a.cost[i] = 0.f;
    a.nvalid[i] = 0u;
    a.last_update[i] = 0u;
}

// Eq. 10 for disc surfels (a disc stays a disc): a usable source surfel (no
// DEGENERATE or UNINIT flag, id_s > 0) moves to p' = R (r_s / id_s) + t with
// n' = R n and is re-centred at u' = K_dst pi(p'), inverse depth 1/p'_z.
// Those with p'_z > 0 and u' in [0, W-1] x [0, H-1] are written in source
// order (as many as there is room for).  One workgroup walks the sources in
// passes of kDiscXferSub chunks of 1024 (a thread's kDiscXferSub landings
// are independent, so their loads and double arithmetic overlap), ranks the
// pass's landings in source order with one scan over (chunk, wavefront)
// and writes them; every landing is computed in double in the oracle's
// order, so the kept set and the order are the same.
//
// Small batches are bound by the host's launches: up to kDiscXferArgs pairs
// travel in the kernel's arguments (4 KB at most), one launch without a table
// upload (six 320x240 pairs, back to back: 6.8 us a call, 13.3 with it).
constexpr int kDiscXferSub = 4;
template <int N>
struct DiscTransferTab {
    DiscTransferArgs pair[N];
};
template <int N>
__global__ __launch_bounds__(1024) void disc_transfer_kernel(DiscTransferTab<N>, const DiscTransferArgs* __restrict__ tab_) {
#pragma clang fp contract(off)
    const cptr<DiscTransferArgs> tab = table_or_arg(tab_);
    const carg<DiscTransferArgs>& a = tab[blockIdx.x];          // one workgroup per keyframe pair
    constexpr int kWaves = 1024 / kWaveSize;
    constexpr int kSlots = kDiscXferSub * kWaves;         // (chunk, wavefront) in source order
    static_assert(kSlots <= kWaveSize, "one wavefront scans the slots");
    __shared__ int s_cnt[kSlots + 1];
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    int base = 0;
    for (int c0 = 0; c0 < a.count; c0 += 1024 * kDiscXferSub) {
        bool land[kDiscXferSub];
        float fu[kDiscXferSub], fv[kDiscXferSub], fid[kDiscXferSub];
        float f0[kDiscXferSub], f1[kDiscXferSub], f2[kDiscXferSub];
        int below[kDiscXferSub];
#pragma unroll
        for (int j = 0; j < kDiscXferSub; ++j) {
            const int k = c0 + j * 1024 + (int)threadIdx.x;
            land[j] = false;
            double u = 0.0, v = 0.0, idn = 0.0, m0 = 0.0, m1 = 0.0, m2 = 0.0;
            if (k < a.count && !(a.flags[k] & (F_DEGENERATE | F_UNINIT)) && a.inv_depth[k] > 0.f) {
                const double ids = a.inv_depth[k];
                const double rs0 = ((double)a.ux[k] - a.sK[2]) / a.sK[0];
                const double rs1 = ((double)a.uy[k] - a.sK[3]) / a.sK[1];
                const double p0 = rs0 / ids, p1 = rs1 / ids, p2 = 1.0 / ids;
                const double n0 = a.nx[k], n1 = a.ny[k], n2 = a.nz[k];
                const double q0 = a.R[0] * p0 + a.R[1] * p1 + a.R[2] * p2 + a.t[0];
                const double q1 = a.R[3] * p0 + a.R[4] * p1 + a.R[5] * p2 + a.t[1];
                const double q2 = a.R[6] * p0 + a.R[7] * p1 + a.R[8] * p2 + a.t[2];
                m0 = a.R[0] * n0 + a.R[1] * n1 + a.R[2] * n2;
                m1 = a.R[3] * n0 + a.R[4] * n1 + a.R[5] * n2;
                m2 = a.R[6] * n0 + a.R[7] * n1 + a.R[8] * n2;
                if (q2 > 0.0) {
                    u = a.dK[0] * (q0 / q2) + a.dK[2];
                    v = a.dK[1] * (q1 / q2) + a.dK[3];
                    land[j] = u >= 0.0 && u <= (double)(a.dst_w - 1) && v >= 0.0 && v <= (double)(a.dst_h - 1);
                    idn = 1.0 / q2;
                }
            }
            // the stored values (rounded to float here rather than at the store)
            fu[j] = (float)u; fv[j] = (float)v; fid[j] = (float)idn;
            f0[j] = (float)m0; f1[j] = (float)m1; f2[j] = (float)m2;
            const unsigned long long ball = __ballot(land[j]);
            below[j] = __popcll(ball & ((1ull << lane) - 1ull));
            if (lane == 0) s_cnt[j * kWaves + wave] = __popcll(ball);
        }
        __syncthreads();
        if (wave == 0) {
            // exclusive scan of the slot counts (slot = lane), total in s_cnt[kSlots]
            const int c = lane < kSlots ? s_cnt[lane] : 0;
            int incl = c;
#pragma unroll
            for (int d = 1; d < kWaveSize; d <<= 1) {
                const int t = __shfl_up(incl, d);
                if (lane >= d) incl += t;
            }
            if (lane < kSlots) s_cnt[lane] = incl - c;
            if (lane == kWaveSize - 1) s_cnt[kSlots] = incl;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kDiscXferSub; ++j) {
            const int k = c0 + j * 1024 + (int)threadIdx.x;
            const int rank = base + s_cnt[j * kWaves + wave] + below[j];
            if (land[j] && rank < a.capacity) {
                a.dst.inv_depth[rank] = fid[j];
                a.dst.nx[rank] = f0[j];
                a.dst.ny[rank] = f1[j];
                a.dst.nz[rank] = f2[j];
                a.dst.flags[rank] = 0u;
                a.dst.cost[rank] = 0.f;
                a.dst.nvalid[rank] = 0u;
                a.dst.last_update[rank] = a.last_update[k];
                a.dux[rank] = fu[j];
                a.duy[rank] = fv[j];
                if (a.src_index) a.src_index[rank] = k;
            }
        }
        base += s_cnt[kSlots];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.counts[0] = min(base, a.capacity);
        a.counts[1] = base;
    }
}

hipError_t launch_disc_transfer(const DiscTransferArgs* pairs, const DiscTransferArgs* table, int n_pairs,
                                hipStream_t s) {
    static_assert(sizeof(DiscTransferTab<kDiscXferArgs>) + sizeof(table) <= 4096, "kernel arguments");
    if (table || n_pairs == 1) {
        disc_transfer_kernel<1><<<n_pairs, 1024, 0, s>>>(DiscTransferTab<1>{{pairs[0]}}, table);
    } else {
        DiscTransferTab<kDiscXferArgs> t;
        std::copy(pairs, pairs + n_pairs, t.pair);
        std::fill(t.pair + n_pairs, t.pair + kDiscXferArgs, DiscTransferArgs{});
        disc_transfer_kernel<kDiscXferArgs><<<n_pairs, 1024, 0, s>>>(t, nullptr);
    }
    return hipGetLastError();
}

template <typename T, bool R>
static void* disc_gn_pick(const DiscForm& f) {
    constexpr int SPW = disc_surfels_per_wave(std::is_same<T, float>::value ? 0 : 1);
    if (f.shared) return (void*)&disc_gn_kernel<T, SPW, R, 1, 2, true>;
    return f.waves == 16  ? (void*)&disc_gn_kernel<T, SPW, R, 16, 4, false>
           : f.waves == 8 ? (void*)&disc_gn_kernel<T, SPW, R, 8, 4, false>
           : f.waves == 4 ? (void*)&disc_gn_kernel<T, SPW, R, 4, 4, false>
           : f.deep == 4  ? (void*)&disc_gn_kernel<T, SPW, R, 1, 4, false>
           : f.deep == 2  ? (void*)&disc_gn_kernel<T, SPW, R, 1, 2, false>
                          : (void*)&disc_gn_kernel<T, SPW, R, 1, 0, false>;
}
template <bool R>
static void* disc_gn_ptr(int dtype, const DiscForm& f) {
    return dtype == 0 ? disc_gn_pick<float, R>(f) : dtype == 1 ? disc_gn_pick<_Float16, R>(f)
                                                               : disc_gn_pick<uint8_t, R>(f);
}

hipError_t launch_disc_gn(int dtype, const DiscForm& form, const LoneBatch& one, const BatchHeader* hdr,
                          int total_items, int grid_blocks, bool by_row, float max_radius, int max_nbr, hipStream_t s,
                          hipEvent_t start, hipEvent_t stop) {
    if (total_items <= 0) return hipSuccess;
    // the unit squares about a disc's pixels lie within radius r + sqrt(1/2)
    const int spw = disc_surfels_per_wave(dtype), lanes = kWaveSize / spw;
    const double reach = (double)max_radius + 0.7072;
    int max_slots = std::min((int)(3.1416 * reach * reach) / lanes + 1, kDiscPPL * spw);
    constexpr int wpb = kBlockThreads / kWaveSize;
    const int lds = form.shared ? wpb * 4 * (spw * max_nbr * kPairWords +
                                             max_slots * kWaveSize * (dtype != 0 ? 1 : 2))
                                : 0;
    void* args[] = {(void*)&one, (void*)&hdr, (void*)&total_items, (void*)&max_slots, (void*)&max_nbr};
    return launch_timed(by_row ? disc_gn_ptr<true>(dtype, form) : disc_gn_ptr<false>(dtype, form), grid_blocks,
                        disc_threads(form.waves), args, s, start, stop, lds);
}

hipError_t launch_disc_render(const DiscRenderItem& one, const DiscRenderItem* table, int n_items,
                              int total_surfels, int total_tiles, bool bin_lds, int px, const DiscRenderScratch& w,
                              hipStream_t s) {
    if (bin_lds) {
        disc_bin_lds_kernel<<<n_items, 1024, 0, s>>>(one, table, w.rec, w.count, w.start, w.list);
    } else {
        // the list's cursor follows the counts
        fill_int_kernel<<<std::min(total_tiles / 256 + 1, 4096), 256, 0, s>>>(w.count, total_tiles + 1, 0);
        const int sblocks = (total_surfels + 255) / 256;
        if (total_surfels > 0)
            disc_count_kernel<<<sblocks, 256, 0, s>>>(one, table, n_items, total_surfels, w.rec, w.count);
        disc_range_kernel<<<(total_tiles + 1023) / 1024, 1024, 0, s>>>(w.count, w.start, w.count + total_tiles, total_tiles);
        if (total_surfels > 0)
            disc_fill_kernel<<<sblocks, 256, 0, s>>>(one, table, n_items, total_surfels, w.rec, w.start, w.list);
    }
    constexpr int wpb = kBlockThreads / kWaveSize;
    const int waves = total_tiles * (4 / px);
    auto* f = px == 1 ? disc_raster_kernel<1> : disc_raster_kernel<4>;
    f<<<(waves + wpb - 1) / wpb, kBlockThreads, 0, s>>>(one, table, n_items, total_tiles, w.rec, w.count, w.start, w.list);
    return hipGetLastError();
}

template <int N>
static hipError_t launch_place(const DiscPlaceTab<N>& by_value, const DiscPlaceArgs* table, int n_items,
                               int total_cands, int total_init, bool small, hipStream_t s) {
    const int waves = kBlockThreads / kWaveSize;
    if (total_cands > 0)
        disc_search_kernel<N><<<(total_cands + waves - 1) / waves, kBlockThreads, 0, s>>>(by_value, table, n_items,
                                                                                           total_cands);
    disc_compact_kernel<N><<<n_items, 1024, 0, s>>>(by_value, table);
    auto* init = small ? disc_init_kernel<N, 2> : disc_init_kernel<N, 9>;
    if (total_init > 0) init<<<total_init, kWaveSize, 0, s>>>(by_value, table, n_items);
    return hipGetLastError();
}

hipError_t launch_disc_place(const DiscPlaceArgs* items, const DiscPlaceArgs* table, int n_items,
                             int total_cands, int total_init, bool small, hipStream_t s) {
    static_assert(sizeof(DiscPlaceTab<kDiscPlaceArgs>) + sizeof(table) + 8 <= 4096, "kernel arguments");
    if (table || n_items == 1)
        return launch_place(DiscPlaceTab<1>{{items[0]}}, table, n_items, total_cands, total_init, small, s);
    DiscPlaceTab<kDiscPlaceArgs> t;
    std::copy(items, items + n_items, t.item);
    std::fill(t.item + n_items, t.item + kDiscPlaceArgs, DiscPlaceArgs{});
    return launch_place(t, nullptr, n_items, total_cands, total_init, small, s);
}

}  // namespace sgn
