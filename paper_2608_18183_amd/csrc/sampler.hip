// Sampling side of a round: the distribution transform of every verifier row,
// probabilistic (Sec. 4.2, Eq. 5) or greedy (Eq. 4) verification of each
// image's window, commit, and the Jacobi window refresh (reused predictions
// first, history tokens at offset H for the rest; Sec. 4.2).
//
// Every fp32 sum over the vocabulary is associated the same way: sequential
// inside consecutive 64-entry chunks, then the chunk totals sequential. The
// inverse CDF returns the first entry whose prefix (chunk prefix plus in-chunk
// prefix) exceeds u * total. Contraction is off in this file so each operation
// rounds once.
#include <type_traits>

#include "common.h"
#include "launch.h"

#pragma clang fp contract(off)

namespace hbsjd {

constexpr int kBins = 1024;     // histogram bins of the top-k threshold search
constexpr int kCand = 256;      // candidates ranked exactly once the bin is this small

// an order-preserving integer image of a float (exact LDS min/max of floats), and back
__device__ inline int float_key(float f) {
    const int i = __builtin_bit_cast(int, f);
    return i >= 0 ? i : i ^ 0x7fffffff;
}
__device__ inline float key_float(int k) {
    return __builtin_bit_cast(float, k >= 0 ? k : k ^ 0x7fffffff);
}

// ---------------------------------------------------------------- transform
// One block per distribution row, two threads per 64-entry chunk: thread t
// holds entries 32 t .. 32 t + 31 in registers, NW wavefronts of 2048 entries
// (8 at V = 16384), so that the per-entry work of a row, some 60 instructions
// an entry, spreads over all four SIMDs of a CU twice. What is left is latency:
// the chains over the chunk sums (about 5000 cycles each) and the block-wide
// phases between them; two blocks of 8 wavefronts share a CU (128 VGPRs; at
// 102 and 80 the code spills or serialises: 43 and 45 us against 40 below).
// With one thread per chunk and single-thread chains, against this, at
// V = 16384: 544 rows, top-k 2000, 49.3 -> 40.9 us; 32 rows 31.3 -> 17.7;
// 1088 rows 76.9 -> 60.0; 4224 guided rows, top-k 1000, 256.7 -> 204.6
// (4.1 TB/s); 20 rows of V = 256 19.6 -> 7.6. A chunk's sum is one chain of
// 64 additions: the even thread's half, handed to the odd thread by a lane
// exchange.
// Global memory is read and written in 1 KB wavefront accesses and transposed
// through the wavefront's own LDS (no block barriers), half of its lanes at a
// time; guidance is combined before that, in the order the rows are read.
constexpr int kTrE = 32;                 // entries per thread
constexpr int kTrStride = kTrE + 4;      // padded so the owners' 16-byte accesses fall in distinct banks

// the calling wavefront's LDS accesses are done (and stay on their side)
__device__ __forceinline__ void wave_lds_sync() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// the value of the even lane of a lane pair, in both lanes (DPP quad permutation [0, 0, 2, 2])
__device__ __forceinline__ float even_lane(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xA0, 0xF, 0xF, false));
}

// The sum of a chunk's 64 values in the pinned order, v the calling thread's
// half: exact in the odd lane of the pair (the even lane returns a partial).
__device__ __forceinline__ float pair_chunk_sum(const float (&v)[kTrE]) {
    float lo = 0.f;
#pragma unroll
    for (int k = 0; k < kTrE; ++k) lo = lo + v[k];
    float s = even_lane(lo);
#pragma unroll
    for (int k = 0; k < kTrE; ++k) s = s + v[k];
    return s;
}

// A wavefront's reduction of an order-free operation by DPP (row shifts, then
// row broadcasts): a tenth of the latency of six LDS exchanges. Uniform result.
template <int Ctrl, int RowMask>
__device__ __forceinline__ int dpp_or_own(int v) {
    return __builtin_amdgcn_update_dpp(v, v, Ctrl, RowMask, 0xF, false);
}
template <typename F>
__device__ __forceinline__ int wave_dpp(int v, F op) {
    v = op(v, dpp_or_own<0x111, 0xF>(v));   // row_shr 1, 2, 4, 8
    v = op(v, dpp_or_own<0x112, 0xF>(v));
    v = op(v, dpp_or_own<0x114, 0xF>(v));
    v = op(v, dpp_or_own<0x118, 0xF>(v));
    v = op(v, dpp_or_own<0x142, 0xA>(v));   // row_bcast 15, 31
    v = op(v, dpp_or_own<0x143, 0xC>(v));
    return __builtin_amdgcn_readlane(v, 63);
}
__device__ __forceinline__ float wave_fmax_dpp(float v) {
    return __int_as_float(wave_dpp(__float_as_int(v), [](int p, int q) {
        return __float_as_int(fmaxf(__int_as_float(p), __int_as_float(q)));
    }));
}
__device__ __forceinline__ float wave_fmin_dpp(float v) {
    return __int_as_float(wave_dpp(__float_as_int(v), [](int p, int q) {
        return __float_as_int(fminf(__int_as_float(p), __int_as_float(q)));
    }));
}
__device__ __forceinline__ int wave_imin_dpp(int v) {
    return wave_dpp(v, [](int p, int q) { return min(p, q); });
}
__device__ __forceinline__ int wave_imax_dpp(int v) {
    return wave_dpp(v, [](int p, int q) { return max(p, q); });
}

// The running sums, from zero and in order, of up to 256 values held four to a
// lane (lane l: values 4 l .. 4 l + 3), by one whole wavefront: each step adds
// a lane's four values to the last sum of the lane below, so the sums of lane
// l are final after l + 1 steps and later steps repeat them. 256 additions in
// a chain without an LDS access between them: a single thread that read the
// values from LDS and wrote the sums there took 6600 cycles, reading alone
// 4800.
__device__ __forceinline__ float4 wave_running_sums(const float4& x, int steps) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int i = 0; i < steps; ++i) {
        // wave_shr 1, zero into lane 0
        const float below = __int_as_float(
            __builtin_amdgcn_update_dpp(0, __float_as_int(v.w), 0x138, 0xF, 0xF, true));
        v.x = below + x.x;
        v.y = v.x + x.y;
        v.z = v.y + x.z;
        v.w = v.z + x.w;
    }
    return v;
}

// f(number of wavefronts that hold a row of V entries)
template <typename F>
static void by_vocab(int V, F f) {
    if (V <= 2048) f(std::integral_constant<int, 1>{});
    else if (V <= 4096) f(std::integral_constant<int, 2>{});
    else if (V <= 8192) f(std::integral_constant<int, 4>{});
    else f(std::integral_constant<int, 8>{});
}

template <int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NW == 8 ? 4 : 3)))
void k_transform(TransformArgs a) {
    constexpr int NT = 64 * NW, E = kTrE;
    __shared__ float redx[NW], redn[NW];
    __shared__ int ired[NW];
    __shared__ int hist[kBins];
    // chunk sums, and their running sums (0 past the row's chunks)
    __shared__ __attribute__((aligned(16))) float tot[NW * 32], pre[NW * 32];
    __shared__ __attribute__((aligned(16))) float cand[kCand];
    __shared__ int s_int[4];
    __shared__ int s_mm[2];
    __shared__ float s_flt[4];
    __shared__ __attribute__((aligned(16))) float stage[NW * 32 * kTrStride];

    const int r = blockIdx.x;
    const bool rows = a.row_pos != nullptr;   // explicit rows
    if (!rows && r >= min(*a.nout_dev, a.nout_cap)) return;
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int V = a.V;
    const int nC = (V + kChunk - 1) / kChunk;
    const int s = r / a.rows_per_slot, i = r - s * a.rows_per_slot;
    const int b = rows ? r : a.slot_img[s];
    const float tau = a.temperature[b];
    // the draw below needs the image's cursor and the seed: fetched now, with
    // the row, rather than after the reductions
    const int pos = rows ? min(max(a.row_pos[r], 0), a.T) : min(a.cursor[b], a.T) + i + 1;
    const uint64_t seed = rows ? ((uint64_t)a.seed_hi << 32) | a.seed_lo : meta_seed(a.meta);
    const float u_draft = uniforms_at(seed, b, pos).draft;
    const float* lc = a.logits + (size_t)((s * a.cfg) * a.rows_per_slot + i) * V;
    const int v0 = t * E;
    float* sw = stage + wv * 32 * kTrStride;

    // the row (entries past V re-read its last float4: unconditional loads stay
    // in flight together), guided, then transposed to its owners
    float y[E];
    {
        const float* lu = a.cfg == 2 ? lc + (size_t)a.rows_per_slot * V : lc;
        bool nan_seen = false;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float4 x[4], w[4];
            const int e0 = wv * 2048 + h * 1024 + 4 * lane;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int v = e0 + q * 256;
                x[q] = *reinterpret_cast<const float4*>(lc + (v < V ? v : V - 4));
            }
            if (a.cfg == 2) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int v = e0 + q * 256;
                    w[q] = *reinterpret_cast<const float4*>(lu + (v < V ? v : V - 4));
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x[q].x = w[q].x + a.cfg_scale * (x[q].x - w[q].x);
                    x[q].y = w[q].y + a.cfg_scale * (x[q].y - w[q].y);
                    x[q].z = w[q].z + a.cfg_scale * (x[q].z - w[q].z);
                    x[q].w = w[q].w + a.cfg_scale * (x[q].w - w[q].w);
                }
            }
            // a NaN logit is an error; entries past V become NaN, which every
            // comparison below rejects
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool in = e0 + q * 256 < V;
                nan_seen |= in && (x[q].x != x[q].x || x[q].y != x[q].y || x[q].z != x[q].z ||
                                   x[q].w != x[q].w);
                const float nan = __builtin_nanf("");
                const int e = q * 256 + 4 * lane;
                *reinterpret_cast<float4*>(sw + (e >> 5) * kTrStride + (e & 31)) =
                    in ? x[q] : make_float4(nan, nan, nan, nan);
            }
            wave_lds_sync();
            if ((lane >> 5) == h) {
                const float* mine = sw + (lane & 31) * kTrStride;
#pragma unroll
                for (int k = 0; k < E; k += 4) {
                    const float4 q4 = *reinterpret_cast<const float4*>(mine + k);
                    y[k] = q4.x;
                    y[k + 1] = q4.y;
                    y[k + 2] = q4.z;
                    y[k + 3] = q4.w;
                }
            }
            wave_lds_sync();
        }
        if (nan_seen) {
            if (rows) *a.err = kErrNanLogit;
            else atomicOr(&a.meta[kMetaError], (int)kErrNanLogit);
        }
    }
    // Max and its lowest index, and min, of the guided logits. Rounding a
    // quotient by tau > 0 keeps order, so those of y are their quotients.
    float ymax, ymin;
    {
        float lmax = -INFINITY, lmin = INFINITY;
        int lidx = 0x7fffffff;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            if (y[k] > lmax) { lmax = y[k]; lidx = k; }
            lmin = fminf(lmin, y[k]);
        }
        const float wmax = wave_fmax_dpp(lmax);
        const float wmin = wave_fmin_dpp(lmin);
        const int widx = wave_imin_dpp(lmax == wmax && lidx < E ? v0 + lidx : 0x7fffffff);
        if (lane == 0) { redx[wv] = wmax; redn[wv] = wmin; ired[wv] = widx; }
        __syncthreads();
        float m = redx[0], mn = redn[0];
        int idx = ired[0];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            if (redx[w] > m) { m = redx[w]; idx = ired[w]; }   // wavefronts hold ascending entries
            mn = fminf(mn, redn[w]);
        }
        if (t == 0) a.amax[r] = idx;
        ymax = m / tau;
        ymin = mn / tau;
    }
    if (tau != 1.0f) {   // x / 1 is x
#pragma unroll
        for (int k = 0; k < E; ++k) y[k] = y[k] / tau;
    }

    // top-k threshold: the k-th largest y counting ties (exact)
    float thr = -INFINITY;
    if (a.top_k > 0 && a.top_k < V) {
        constexpr int BPT = kBins / NT;   // bins per thread in the scan
        float lo = ymin, hi = ymax;
        int above = 0;   // entries strictly above the current range
        for (int iter = 0; iter < 64; ++iter) {
            if (lo == hi) { thr = lo; break; }
#pragma unroll
            for (int q = 0; q < BPT; ++q) hist[t + NT * q] = 0;
            __syncthreads();
            const float scale = (float)kBins / (hi - lo);
            // the bins are kept, two to a register, for the passes below
            // (out of range: a bin that is never chosen)
            uint32_t bins[E / 2];
            auto count = [&](int k, bool in, uint32_t bin) {
                bins[k / 2] = k & 1 ? bins[k / 2] | bin << 16 : bin;
                if (in) atomicAdd(&hist[bin], 1);
            };
            if (__builtin_expect(scale > 0.f && scale < INFINITY, 1)) {
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    const float yy = y[k];
                    const bool in = yy >= lo && yy <= hi;
                    count(k, in, in ? (uint32_t)min((int)((yy - lo) * scale), kBins - 1) : 0xFFFFu);
                }
            } else {
                // the range has no finite width (masked entries at -inf, a
                // difference that overflows) or too small a one to divide by:
                // bins of equal width on the order-preserving integer image
                // instead, in which any range splits. The additions make -0
                // +0, and `nil` keeps them inside the search loop. (That this
                // path is there costs a launch that does not take it 0.5%:
                // 232.6 -> 233.8 us with 4224 guided rows of 16384; halving the
                // range there, shorter code, cost 2%.)
                float nil = 0.f;
                asm volatile("" : "+v"(nil));
                const uint32_t first = (uint32_t)float_key(lo + nil);
                const uint32_t width = (uint32_t)float_key(hi + nil) - first;
                const int shift = max(22 - __clz((int)width), 0);   // the top ten bits
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    const float yy = y[k];
                    const bool in = yy >= lo && yy <= hi;
                    const uint32_t bin = ((uint32_t)float_key(yy + nil) - first) >> shift;
                    count(k, in, in ? min(bin, (uint32_t)kBins - 1) : 0xFFFFu);
                }
            }
            __syncthreads();
            // suffix counts: thread t owns bins BPT t .. BPT t + BPT - 1
            int own = 0;
#pragma unroll
            for (int q = 0; q < BPT; ++q) own += hist[BPT * t + q];
            // inclusive suffix scan over threads (higher threads = higher bins)
            int sfx = own;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int yv = __shfl_down(sfx, o, 64);
                if (lane + o < 64) sfx += yv;
            }
            if (lane == 0) ired[wv] = sfx;
            if (t == 0) {
                s_int[0] = -1;
                s_int[1] = 0;
                s_int[2] = 0;
                s_int[3] = 0;
                s_mm[0] = 0x7fffffff;
                s_mm[1] = (int)0x80000000;
            }
            __syncthreads();
            for (int w = wv + 1; w < NW; ++w) sfx += ired[w];
            // entries in bins above thread t's group
            int cum = above + sfx - own;
            for (int q = BPT - 1; q >= 0; --q) {
                const int hb = hist[BPT * t + q];
                if (cum < a.top_k && a.top_k <= cum + hb) {
                    s_int[0] = BPT * t + q;
                    s_int[1] = cum;
                    s_int[2] = hb;
                }
                cum += hb;
            }
            __syncthreads();
            const int bstar = s_int[0];
            const int above_new = s_int[1];
            const int cnt = s_int[2];
            if (bstar < 0) {   // only with NaN logits, which are reported as an error
                thr = lo;
                break;
            }
            if (cnt <= kCand) {
                uint32_t mine = 0;
#pragma unroll
                for (int k = 0; k < E; ++k)
                    mine |= (uint32_t)((k & 1 ? bins[k / 2] >> 16 : bins[k / 2] & 0xFFFFu) ==
                                       (uint32_t)bstar) << k;
                // one reservation per thread, not one per candidate
                if (mine) {
                    int slot = atomicAdd(&s_int[3], __popc(mine));
#pragma unroll
                    for (int k = 0; k < E; ++k)
                        if (mine >> k & 1) cand[slot++] = y[k];
                }
                __syncthreads();
                const int need = a.top_k - above_new;   // rank inside the bin, 1-based
                for (int c = t; c < cnt; c += NT) {
                    const float cv = cand[c];
                    int gt = 0, ge = 0;
#pragma unroll 8
                    for (int j = 0; j < cnt; ++j) {
                        gt += cand[j] > cv;
                        ge += cand[j] >= cv;
                    }
                    if (gt < need && need <= ge) s_flt[0] = cv;
                }
                __syncthreads();
                thr = s_flt[0];
                break;
            }
            // narrow to the values that fell into the chosen bin: their exact
            // minimum and maximum, on an order-preserving integer image of the
            // float: per thread (chains cut every 8 entries, so the compiler
            // does not rebalance them into trees), per wavefront, then across
            // the block through LDS atomics. The images are formed from a
            // copy of the entries the compiler cannot see through, so it does
            // not hoist all of them out of the search loop
            {
                int zero = 0;
                asm volatile("" : "+v"(zero));
                int mn = 0x7fffffff, mx = (int)0x80000000;
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    if ((k & 7) == 0) asm volatile("" : "+v"(mn), "+v"(mx));
                    const bool sel = (k & 1 ? bins[k / 2] >> 16 : bins[k / 2] & 0xFFFFu) ==
                                     (uint32_t)bstar;
                    const int bits = __float_as_int(y[k]) | zero;
                    const int key = bits >= 0 ? bits : bits ^ 0x7fffffff;
                    mn = sel && key < mn ? key : mn;
                    mx = sel && key > mx ? key : mx;
                }
                mn = wave_imin_dpp(mn);
                mx = wave_imax_dpp(mx);
                if (lane == 0) {
                    atomicMin(&s_mm[0], mn);
                    atomicMax(&s_mm[1], mx);
                }
            }
            __syncthreads();
            lo = key_float(s_mm[0]);
            hi = key_float(s_mm[1]);
            __syncthreads();
            above = above_new;
            thr = lo;   // only reached if the loop runs out: keeps at least k entries
        }
    }

    // softmax over the kept entries; Z in the pinned chunk order
#pragma unroll
    for (int k = 0; k < E; ++k) y[k] = (y[k] >= thr) ? expf(y[k] - ymax) : 0.f;
    {
        const float csum = pair_chunk_sum(y);
        if (t & 1) tot[t >> 1] = csum;
    }
    __syncthreads();
    const int csteps = (nC + 3) >> 2;   // lanes that hold chunk sums
    const int cl = min(4 * lane, NW * 32 - 4);
    if (wv == 0) {
        const float4 c = wave_running_sums(*reinterpret_cast<const float4*>(tot + cl), csteps);
        if (lane == csteps - 1) s_flt[1] = c.w;   // sums past the row's chunks are 0
        if (t == 0) s_int[2] = -1;   // the row's last positive entry, gathered below
    }
    __syncthreads();
    const float z = s_flt[1];
    // p = e / z, correctly rounded. While every kept e is at least 2^-80 (its
    // remainders are then exact) and 1 <= z, the quotient comes from the
    // rounded reciprocal by two residual corrections (the first leaves it
    // within an ulp, and a remainder's correction of such a quotient rounds
    // correctly: Markstein, IBM J. Res. Dev. 34, 1990): five operations
    // against the eleven of a division that scales its operands.
    const float lowest = thr > ymin ? thr : ymin;
    if (lowest - ymax > -55.f && z >= 1.f) {
        const float rz = 1.0f / z;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            const float e = y[k];
            float q = e * rz;
            q = __builtin_fmaf(__builtin_fmaf(-q, z, e), rz, q);
            y[k] = __builtin_fmaf(__builtin_fmaf(-q, z, e), rz, q);
        }
    } else {
#pragma unroll
        for (int k = 0; k < E; ++k) y[k] = y[k] / z;
    }
    uint32_t pos_mask = 0;   // entries past V are 0, so never positive
#pragma unroll
    for (int k = 0; k < E; ++k) pos_mask |= (uint32_t)(y[k] > 0.f) << k;
    // this thread's last positive entry (the fallback of the draw below)
    const int last_pos = pos_mask ? v0 + 31 - __clz((int)pos_mask) : -1;
    {
        const float psum = pair_chunk_sum(y);
        if (t & 1) tot[t >> 1] = psum;
        const int lw = wave_imax_dpp(last_pos);
        if (lane == 0) atomicMax(&s_int[2], lw);
    }
    // one wavefront runs the prefix while the others store the row
    __syncthreads();
    if (wv == 0) {
        const float4 c = wave_running_sums(*reinterpret_cast<const float4*>(tot + cl), csteps);
        if (4 * lane < NW * 32) *reinterpret_cast<float4*>(pre + 4 * lane) = c;
    }
    float* prow = a.p + (size_t)r * V;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if ((lane >> 5) == h) {
            float* mine = sw + (lane & 31) * kTrStride;
#pragma unroll
            for (int k = 0; k < E; k += 4)
                *reinterpret_cast<float4*>(mine + k) = make_float4(y[k], y[k + 1], y[k + 2], y[k + 3]);
        }
        wave_lds_sync();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = q * 256 + 4 * lane;
            const int v = wv * 2048 + h * 1024 + e;
            const float4 x = *reinterpret_cast<const float4*>(sw + (e >> 5) * kTrStride + (e & 31));
            if (v < V) *reinterpret_cast<float4*>(prow + v) = x;
        }
        wave_lds_sync();
    }
    __syncthreads();

    // draft candidate of this row: the position it predicts is n_b + i + 1 no
    // matter how the round's verification ends, so its draw from p with
    // u_draft(b, n_b + i + 1) is taken here, with the row's own prefix: the
    // same sums and search as block_draw over the stored row, hence
    // the same token. The running sums of non-negative values never fall, so
    // the first one above the target is as many as lie at or below it.
    if (pos > a.T) {
        if (t == 0) a.samp[r] = -1;
        return;
    }
    const float target = u_draft * pre[nC - 1];
    int cs = -1;   // every wavefront finds the chunk for itself
#pragma unroll
    for (int c0 = (NW * 32 - 1) / 64 * 64; c0 >= 0; c0 -= 64) {
        const int c = c0 + lane;
        const uint64_t above = __ballot(c < nC && pre[min(c, NW * 32 - 1)] > target);
        if (above) cs = c0 + __ffsll((unsigned long long)above) - 1;
    }
    if (cs < 0) {   // rounding left the target above the total, or no entry is positive
        if (t == 0) {
            a.samp[r] = s_int[2];
            if (a.amax[r] >= V) a.amax[r] = 0;   // no entry above -inf: the first
        }
        return;
    }
    if ((t >> 1) != cs) return;
    // the chunk's two owners walk it in order
    const float before = cs > 0 ? pre[cs - 1] : 0.f;
    float inner = 0.f;
    int n0 = 0, n1 = 0;
#pragma unroll
    for (int k = 0; k < E; ++k) {
        inner = inner + y[k];
        n0 += before + inner > target ? 0 : 1;
    }
    inner = even_lane(inner);
    n0 = __float_as_int(even_lane(__int_as_float(n0)));
    const int last0 = __float_as_int(even_lane(__int_as_float(last_pos)));
#pragma unroll
    for (int k = 0; k < E; ++k) {
        inner = inner + y[k];
        n1 += before + inner > target ? 0 : 1;
    }
    if (t & 1) {
        const int n = n0 < E ? n0 : E + n1;
        a.samp[r] = n < kChunk ? cs * kChunk + n : last_pos >= 0 ? last_pos : last0;
    }
}

void transform(const TransformArgs& a, hipStream_t s) {
    if (a.nout_cap <= 0) return;
    by_vocab(a.V, [&](auto nw) {
        constexpr int NW = decltype(nw)::value;
        launch(k_transform<NW>, dim3(a.nout_cap), dim3(64 * NW), 0, s, a);
    });
}

// ---------------------------------------------------------------- replacement draw
// LDS of one block's replacement draw
template <int NW>
struct DrawLds {
    __attribute__((aligned(16))) float stage[NW * 32 * kTrStride];
    __attribute__((aligned(16))) float tot[NW * 32], pre[NW * 32];   // chunk sums, running sums
    int last, res;
};

// Block-level inverse CDF over non-negative weights, thread t holding entries
// 32 t .. 32 t + 31 (0 past V), in the pinned association: the first entry
// whose chunk prefix plus in-chunk prefix exceeds u * total, else the last
// positive entry. Returns -1 when every weight is zero. Every thread of the
// block's NW wavefronts must call it.
template <int NW>
__device__ __forceinline__ int block_draw(const float (&w)[kTrE], int V, float u, DrawLds<NW>& l) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int nC = (V + kChunk - 1) / kChunk;
    if (t == 0) l.last = -1;
    const float sum = pair_chunk_sum(w);
    if (t & 1) l.tot[t >> 1] = sum;
    uint32_t pos_mask = 0;
#pragma unroll
    for (int k = 0; k < kTrE; ++k) pos_mask |= (uint32_t)(w[k] > 0.f) << k;
    const int last_pos = pos_mask ? t * kTrE + 31 - __clz((int)pos_mask) : -1;
    const int lw = wave_imax_dpp(last_pos);
    __syncthreads();
    if (lane == 0) atomicMax(&l.last, lw);
    if (wv == 0) {
        const int cl = min(4 * lane, NW * 32 - 4);
        const float4 c =
            wave_running_sums(*reinterpret_cast<const float4*>(l.tot + cl), (nC + 3) >> 2);
        if (4 * lane < NW * 32) *reinterpret_cast<float4*>(l.pre + 4 * lane) = c;
    }
    __syncthreads();
    const float total = l.pre[nC - 1];
    if (!(total > 0.f)) return -1;
    const float target = u * total;
    // running sums of non-negative values never fall: the first one above the
    // target is as many as lie at or below it
    int cs = -1;   // every wavefront finds the chunk for itself
#pragma unroll
    for (int c0 = (NW * 32 - 1) / 64 * 64; c0 >= 0; c0 -= 64) {
        const int c = c0 + lane;
        const uint64_t above = __ballot(c < nC && l.pre[min(c, NW * 32 - 1)] > target);
        if (above) cs = c0 + __ffsll((unsigned long long)above) - 1;
    }
    if (cs < 0) return l.last;   // rounding left the target above the total
    if ((t >> 1) == cs) {        // the chunk's two owners walk it in order
        const float before = cs > 0 ? l.pre[cs - 1] : 0.f;
        float inner = 0.f;
        int n0 = 0, n1 = 0;
#pragma unroll
        for (int k = 0; k < kTrE; ++k) {
            inner = inner + w[k];
            n0 += before + inner > target ? 0 : 1;
        }
        inner = even_lane(inner);
        n0 = __float_as_int(even_lane(__int_as_float(n0)));
        const int last0 = __float_as_int(even_lane(__int_as_float(last_pos)));
#pragma unroll
        for (int k = 0; k < kTrE; ++k) {
            inner = inner + w[k];
            n1 += before + inner > target ? 0 : 1;
        }
        const int n = n0 < kTrE ? n0 : kTrE + n1;
        if (t & 1) l.res = n < kChunk ? cs * kChunk + n : last_pos >= 0 ? last_pos : last0;
    }
    __syncthreads();
    return l.res;
}

// The replacement token of a rejected draft (Sec. 4.2, Eq. 5): a draw with u
// from the residual max(0, p - q), where q is the proposal row `qrow`, or a
// point mass on z when qrow is null (a history draft); from p itself when the
// residual is zero everywhere in fp32. Rows of up to 2048 NW entries, every
// thread of the block must call. Latency-bound (one block per image): the
// two rows' loads are all in flight together, the residual is formed in the
// order they are read and transposed to its owners once, and the sums run as
// in the transform (B = 128, W = 32, V = 16384: 16.8 -> 9.1 us a launch).
template <int NW>
__device__ __forceinline__ int replacement_draw(const float* __restrict__ pr,
                                                const float* __restrict__ qrow, int z, int V,
                                                float u, DrawLds<NW>& l) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float* sw = l.stage + wv * 32 * kTrStride;
    for (int pass = 0;; ++pass) {   // the second one draws from p
        float4 x[8], y[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int v = wv * 2048 + q * 256 + 4 * lane;
            x[q] = *reinterpret_cast<const float4*>(pr + (v < V ? v : V - 4));
        }
        if (qrow) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int v = wv * 2048 + q * 256 + 4 * lane;
                y[q] = *reinterpret_cast<const float4*>(qrow + (v < V ? v : V - 4));
            }
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int v = wv * 2048 + q * 256 + 4 * lane;
                y[q] = make_float4(v == z ? 1.f : 0.f, v + 1 == z ? 1.f : 0.f,
                                   v + 2 == z ? 1.f : 0.f, v + 3 == z ? 1.f : 0.f);
            }
        }
        float w[kTrE];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = q * 256 + 4 * lane;
                const bool in = wv * 2048 + h * 1024 + e < V;
                auto part = [&](float pv, float qv) {
                    const float d = pass ? pv : pv - qv;
                    return in && d > 0.f ? d : 0.f;
                };
                const float4 pv = x[4 * h + q], qv = y[4 * h + q];
                *reinterpret_cast<float4*>(sw + (e >> 5) * kTrStride + (e & 31)) =
                    make_float4(part(pv.x, qv.x), part(pv.y, qv.y), part(pv.z, qv.z),
                                part(pv.w, qv.w));
            }
            wave_lds_sync();
            if ((lane >> 5) == h) {
                const float* mine = sw + (lane & 31) * kTrStride;
#pragma unroll
                for (int k = 0; k < kTrE; k += 4) {
                    const float4 q4 = *reinterpret_cast<const float4*>(mine + k);
                    w[k] = q4.x;
                    w[k + 1] = q4.y;
                    w[k + 2] = q4.z;
                    w[k + 3] = q4.w;
                }
            }
            wave_lds_sync();
        }
        const int rep = block_draw<NW>(w, V, u, l);
        if (rep >= 0 || pass == 1) return rep;
    }
}

// ---------------------------------------------------------------- verify + commit + refresh
// One block of NW wavefronts (2048 NW >= V) per processed image.
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_verify(VerifyArgs a) {
    __shared__ DrawLds<NW> draw;
    __shared__ int s_first;
    __shared__ int old_dr[64], old_q[64];
    __shared__ int new_dr[64], new_q[64];

    const int sl = blockIdx.x;
    if (sl >= min(*a.nimg_dev, a.nimg_cap)) return;
    const int t = threadIdx.x;
    const int b = a.slot_img[sl];
    const int n = a.cursor[b];
    if (n >= a.T) return;              // finished image in Full mode: rows discarded
    const int W = a.W, V = a.V, R = a.rows_per_slot;
    const uint64_t seed = meta_seed(a.meta);
    if (a.ar) {
        // cached AR: the image's single row predicts position n + 1 (Eq. 1)
        if (t >= 64) return;
        const int prow = sl * R;
        const int z = a.greedy ? a.amax[prow] : a.samp[prow];
        if (t == 0) {
            if (z < 0) atomicOr(&a.meta[kMetaError], (int)kErrNoProbability);
            a.xtok[(size_t)b * a.T + n] = z;
            const int round = a.meta[kMetaRound];
            if (a.counts && round >= 0 && round < a.max_rounds) a.counts[(size_t)round * a.B + b] = 1;
            atomicAdd((unsigned long long*)&a.stats[0], 1ull);
            atomicAdd((unsigned long long*)&a.stats[2], 1ull);
            a.cursor[b] = n + 1;
        }
        return;
    }
    int n_new, base, nrows;
    if (a.prefill) {
        n_new = n;
        base = n;
        nrows = 1;
    } else {
        // the batch-synchronous ablation stops at the image's window end; an
        // image already there verifies nothing and only re-draws its window
        const int We = max(min(W, (a.win_end ? a.win_end[b] : a.T) - n), 0);
        if (t < W) {
            old_dr[t] = a.drafts[(size_t)b * W + t];
            old_q[t] = a.qsrc[(size_t)b * W + t];
        }
        if (t == 0) s_first = We + 1;
        __syncthreads();
        if (t < We) {
            const int j = t + 1;
            const int z = old_dr[t];
            const int prow = sl * R + (j - 1);
            bool acc = false;
            if (a.greedy) {
                acc = z == a.amax[prow];
            } else if (z < 0) {   // the draw of a row without a positive probability
                atomicOr(&a.meta[kMetaError], (int)kErrNoProbability);
            } else {
                const float P = a.p[(size_t)prow * V + z];
                const int qs = old_q[t];
                const float Q = qs >= 0 ? a.p_prev[(size_t)qs * V + z] : 1.0f;
                if (!(Q > 0.f)) atomicOr(&a.meta[kMetaError], (int)kErrZeroProposal);
                const float u = uniforms_at(seed, b, n + j).acc;
                acc = (P >= Q) || (u < P / Q);
            }
            if (!acc) atomicMin(&s_first, j);
        }
        __syncthreads();
        const int js = s_first;
        const bool rejected = js <= We;
        const int count = rejected ? js : We;
        int rep = 0;
        if (rejected) {
            const int prow = sl * R + (js - 1);
            if (a.greedy) {
                rep = a.amax[prow];
            } else {
                const int qs = old_q[js - 1];
                const float u = uniforms_at(seed, b, n + js).res;
                rep = replacement_draw<NW>(a.p + (size_t)prow * V,
                                           qs >= 0 ? a.p_prev + (size_t)qs * V : nullptr,
                                           old_dr[js - 1], V, u, draw);
            }
        }
        // commit x_{n+1..n+count}
        if (t < count) {
            const int tok = (t == count - 1 && rejected) ? rep : old_dr[t];
            a.xtok[(size_t)b * a.T + n + t] = tok;
        }
        if (t == 0) {
            if (rep < 0) atomicOr(&a.meta[kMetaError], (int)kErrNoProbability);
            const int round = a.meta[kMetaRound];
            if (a.counts && round >= 0 && round < a.max_rounds) a.counts[(size_t)round * a.B + b] = count;
            atomicAdd((unsigned long long*)&a.stats[0], (unsigned long long)count);
            atomicAdd((unsigned long long*)&a.stats[1], (unsigned long long)(rejected ? 1 : 0));
            atomicAdd((unsigned long long*)&a.stats[2], count > 0 ? 1ull : 0ull);
            a.cursor[b] = n + count;
        }
        n_new = n + count;
        base = n;
        nrows = We + 1;
        __syncthreads();
    }
    // refresh the window for positions n_new+1 .. n_new+span
    if (n_new >= a.T) {
        if (t < W) {
            a.drafts[(size_t)b * W + t] = -1;
            a.qsrc[(size_t)b * W + t] = -1;
        }
        return;
    }
    const int span = min(W, a.T - n_new);
    const int reused = min(span, base + nrows - n_new);   // positions covered by this round's rows
    // reused predictions: the transform drew each row's candidate for the
    // position it predicts (u_draft of that position), or took its argmax
    for (int m = 1 + t; m <= reused; m += 64 * NW) {
        const int pos = n_new + m;
        const int prow = sl * R + (pos - base - 1);
        new_dr[m - 1] = a.greedy ? a.amax[prow] : a.samp[prow];
        new_q[m - 1] = prow;
    }
    __syncthreads();
    // the rest take the token H back (or one back near the start); a window
    // position that is itself such a token passes on its own source
    for (int m = max(reused, 0) + 1 + t; m <= span; m += 64 * NW) {
        int src = n_new + m;
        do src = src - a.H >= 1 ? src - a.H : src - 1;
        while (src > n_new + max(reused, 0));
        // both candidates are loaded from their own arrays and the value
        // selected, so neither access goes through a generic pointer
        const int from_x = a.xtok[(size_t)b * a.T + max(min(src, n_new) - 1, 0)];
        const int from_w = new_dr[max(src - n_new - 1, 0)];
        new_dr[m - 1] = src <= n_new ? from_x : from_w;
        new_q[m - 1] = -1;
    }
    __syncthreads();
    if (t < W) {
        a.drafts[(size_t)b * W + t] = t < span ? new_dr[t] : -1;
        a.qsrc[(size_t)b * W + t] = t < span ? new_q[t] : -1;
    }
}

void verify_commit(const VerifyArgs& a, hipStream_t s) {
    if (a.nimg_cap <= 0) return;
    by_vocab(a.V, [&](auto nw) {
        constexpr int NW = decltype(nw)::value;
        launch(k_verify<NW>, dim3(a.nimg_cap), dim3(64 * NW), 0, s, a);
    });
}

// ---------------------------------------------------------------- state export
// q[i] = the proposal probability of draft i: its source row's p(z) for a
// reused prediction (qsrc >= 0) in probabilistic mode, 1 for a history draft
// (point mass) or in greedy mode, 0 where there is no draft
__global__ void k_gather_q(const float* __restrict__ P, const int32_t* __restrict__ qsrc,
                           const int32_t* __restrict__ drafts, int n, int V, int greedy,
                           float* __restrict__ q) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int z = drafts[i], qs = qsrc[i];
    float v = 0.f;
    if (z >= 0) v = (greedy || qs < 0) ? 1.0f : P[(size_t)qs * V + z];
    q[i] = v;
}

void gather_q(const float* P, const int32_t* qsrc, const int32_t* drafts, int n, int V,
              int greedy, float* q, hipStream_t s) {
    if (n <= 0) return;
    launch(k_gather_q, dim3((n + 255) / 256), dim3(256), 0, s, P, qsrc, drafts, n, V, greedy, q);
}

// ---------------------------------------------------------------- explicit-row transform
// Metadata of a transform over caller rows: row r is image r at sequence
// position pos[r] (clamped to [0, kRowPosMax]); the row's draw then uses
// u_draft(seed, r, pos[r]).
__global__ void k_transform_rows_setup(int rows, uint32_t seed_lo, uint32_t seed_hi,
                                       const int32_t* __restrict__ pos, int32_t* slot_img,
                                       int32_t* cursor, int32_t* meta) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < rows) {
        slot_img[i] = i;
        cursor[i] = min(max(pos[i], 0), kRowPosMax) - 1;
    }
    if (i < kMetaCount) {
        int v = 0;
        if (i == kMetaOutRows) v = rows;
        if (i == kMetaSeedLo) v = (int32_t)seed_lo;
        if (i == kMetaSeedHi) v = (int32_t)seed_hi;
        meta[i] = v;
    }
}

void transform_rows(int rows, int V, const float* logits, int cfg, float cfg_scale,
                    const float* temperature, int top_k, uint64_t seed, const int32_t* pos,
                    float* p, int32_t* amax, int32_t* draw, int32_t* scratch, hipStream_t s) {
    int32_t* slot_img = scratch;
    int32_t* cursor = scratch + rows;
    int32_t* meta = scratch + 2 * (size_t)rows;
    const int n = rows > kMetaCount ? rows : kMetaCount;
    launch(k_transform_rows_setup, dim3((n + 255) / 256), dim3(256), 0, s, rows, (uint32_t)seed,
           (uint32_t)(seed >> 32), pos, slot_img, cursor, meta);
    TransformArgs a{logits, p, amax, draw, slot_img, cursor, temperature, 1, cfg, V, top_k,
                    kRowPosMax, cfg_scale, meta + kMetaOutRows, rows, meta};
    transform(a, s);
}

void transform_rows_direct(int rows, int V, const float* logits, int cfg, float cfg_scale,
                           const float* temperature, int top_k, uint64_t seed, const int32_t* pos,
                           float* p, int32_t* amax, int32_t* draw, volatile int32_t* err,
                           hipStream_t s) {
    TransformArgs a{logits, p, amax, draw, nullptr, nullptr, temperature, 1, cfg, V, top_k,
                    kRowPosMax, cfg_scale, nullptr, rows, nullptr};
    a.row_pos = pos;
    a.seed_lo = (uint32_t)seed;
    a.seed_hi = (uint32_t)(seed >> 32);
    a.err = err;
    transform(a, s);
}

// ---------------------------------------------------------------- explicit-row verification
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_verify_probs(int W, int V, const float* p,
                                                          const float* q, const int32_t* drafts,
                                                          const float* u_acc, const float* u_res,
                                                          int32_t* counts, int32_t* tokens) {
    __shared__ DrawLds<NW> draw;
    __shared__ int s_first;
    __shared__ int s_bad;
    const int b = blockIdx.x, t = threadIdx.x;
    if (t == 0) {
        s_first = W + 1;
        s_bad = 0;
    }
    __syncthreads();
    for (int j = t; j < W; j += 64 * NW) {
        const int z = drafts[(size_t)b * W + j];
        if (z < 0 || z >= V) s_bad = 1;
    }
    __syncthreads();
    if (s_bad) {
        for (int j = t; j < W; j += 64 * NW) tokens[(size_t)b * W + j] = -1;
        if (t == 0) counts[b] = 0;
        return;
    }
    for (int j = t; j < W; j += 64 * NW) {
        const size_t row = (size_t)b * W + j;
        const int z = drafts[row];
        const float P = p[row * V + z];
        const float Q = q[row * V + z];
        const bool acc = (P >= Q) || (u_acc[row] < P / Q);
        if (!acc) atomicMin(&s_first, j + 1);
    }
    __syncthreads();
    const int js = s_first;
    const bool rejected = js <= W;
    const int count = rejected ? js : W;
    int rep = 0;
    if (rejected) {
        const size_t row = (size_t)b * W + js - 1;
        rep = replacement_draw<NW>(p + row * V, q + row * V, drafts[row], V, u_res[b], draw);
    }
    for (int j = t; j < W; j += 64 * NW) {
        const size_t row = (size_t)b * W + j;
        int tok = -1;
        if (j < count) tok = (j == count - 1 && rejected) ? rep : drafts[row];
        tokens[row] = tok;
    }
    if (t == 0) counts[b] = count;
}

void verify_probs(int B, int W, int V, const float* p, const float* q, const int32_t* drafts,
                  const float* u_acc, const float* u_res, int32_t* counts, int32_t* tokens,
                  hipStream_t s) {
    if (B <= 0) return;
    by_vocab(V, [&](auto nw) {
        constexpr int NW = decltype(nw)::value;
        launch(k_verify_probs<NW>, dim3(B), dim3(64 * NW), 0, s, W, V, p, q, drafts, u_acc, u_res,
               counts, tokens);
    });
}

}  // namespace hbsjd
