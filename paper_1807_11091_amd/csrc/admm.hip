// gfx950 kernels and entry points of the ADMM Z-update (projection onto the
// sparsity sets of Section 3, as solved in Section 4), of the dual update /
// gradient of eq. (3), and of the W-subproblem's SGD step, also used for masked
// retraining (k_sgd).
//
// Data flow of structadmm_project for one dependency level of layers:
//   k_expand_allowed  (channel and shape layers with an input-channel support)
//                     per-column support bytes; the other sets read the mask, an
//                     element-wise layer a copy of it if the level overwrites it
//   k_row_scores      filter sets: one wavefront per weight row, O_a in binary64
//   k_col_partials    channel / shape sets: binary64 column sums per band of rows
//   k_select          one workgroup per structured layer: final scores, radix
//                     select of the k-th largest score bits in LDS, lowest-index
//                     tie-break, mask + ascending kept_idx, per-column keep bytes
//   k_elem_*          non-structured sets: 3 histogram passes over |v| bits, then an
//                     order-preserving count / apply
//   k_apply           flat streaming Z (+ fused U', G) writer over every layer
// Every reduction has a fixed order; no floating-point atomics are used.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <vector>

#include "sa_device.h"
#include "sa_host.h"
#include "structadmm.h"

namespace sa {
namespace {

constexpr int kTab = 64;           // layers per launch (kernel-argument table, < 8 KiB; ResNet-50's
                                   // 53 convolutions take one launch per phase)
constexpr int kRowThreads = 256;   // 4 wavefronts, one weight row each at a time
constexpr int kRowItems = 2;       // work items per wavefront
constexpr int kColThreads = 256;
constexpr int kColBand = 32;       // rows per band of column partial sums
constexpr int kColSlices = 4;      // row slices of a band (one wavefront each)
constexpr int kSelThreads = 1024;
constexpr int kElemThreads = 256;  // count and apply passes
constexpr int kHistThreads = 1024;
constexpr int kElemPerThread = 8;
constexpr int kElemChunk = kElemThreads * kElemPerThread;  // entries per step of a workgroup
constexpr int kHistChunk = kHistThreads * kElemPerThread;
constexpr int kElemMaxBlocks = 1024;  // blocks per layer: a block adds up the counts of those before it
constexpr int kElemTab = 32;          // element-wise layers per launch

// ---------------------------------------------------------------- tables
struct RowLayer {
    const float *W;
    float *U;
    const uint8_t *allowed;  // [groups*K] or null: every entry inside the support
    const uint8_t *inmask;   // [groups*B] or null: filter sets read the support from the
                             // input-channel mask itself (entry (a, j) is inside when
                             // inmask[(a / Ag) * B + j / CD] is set)
    double *scores;          // [A] (row scores)
    double *rowpart;         // [A][nchunk] partial row sums when nchunk > 1
    int32_t A, K, Ag;        // rows, row length, rows per conv group
    int32_t R, nchunk;       // rows per wavefront item (short rows), 1024-weight chunks per row
    int32_t vec;             // K % 4 == 0: float4 path
    int32_t B;               // input channels per conv group (inmask)
    FastDiv divCD;           // taps per channel (inmask)
    float rho;
};
struct RowTab {
    RowLayer L[kTab];
    int32_t begin[kTab + 1];
    int32_t nl;
};

struct ColLayer {
    const float *W;
    const float *U;
    const uint8_t *allowed;
    double *partials;  // [nbands][K]
    int32_t A, K, Ag, nbands, ctiles, vec;
};
struct ColTab {
    ColLayer L[kTab];
    int32_t begin[kTab + 1];
    int32_t nl;
};

struct SelLayer {
    const double *partials;  // channel / shape: [nbands][K]
    const double *rowpart;   // filter with chunked rows: [G][nchunk]
    double *scores;          // [G]: filter: input (or output with rowpart); channel / shape: output
    uint8_t *mask;           // [G]
    int32_t *kept_idx;       // [k]
    uint8_t *colkeep;        // [groups*K] or null
    const uint8_t *allowed;  // [groups*K] or null
    int32_t kind, G, k, K, CD, nbands, groups, nchunk;
};
struct SelTab {
    SelLayer L[kTab];
    int32_t nl;
};

struct DualLayer {
    const float *W;
    const float *Z;
    float *U;
    float *G;
    int32_t n, update;
    float rho;
};
struct DualTab {
    DualLayer L[kTab];
    int32_t begin[kTab + 1];
    int32_t nl;
};

struct SgdLayer {
    float *W;
    const float *Gf;
    const float *Z;
    const float *U;
    const uint8_t *mask;
    int32_t n, kind;
    FastDiv divK, divCD;  // entry -> filter, column -> channel
    float rho, lr;
};
struct SgdTab {
    SgdLayer L[kTab];
    int32_t begin[kTab + 1];
    int32_t nl;
};

__device__ inline int find_layer(const int32_t *begin, int nl, int b) {
    // the last layer whose first block is at or below b (binary search: a
    // launch holds up to 64 layers)
    int lo = 0, hi = nl - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (begin[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Stores 4 consecutive binary32 values (16-byte aligned) with the
// non-temporal hint: streamed output that nothing reads back soon.
typedef float f32x4v __attribute__((ext_vector_type(4)));
__device__ inline void nt_store4(float *p, const float *v) {
    __builtin_nontemporal_store(f32x4v{v[0], v[1], v[2], v[3]}, reinterpret_cast<f32x4v *>(p));
}

// ---------------------------------------------------------------- support
// allowed[gc*K + j] = in_ch_mask[gc*B + j / CD]
__global__ void k_expand_allowed(const uint8_t *__restrict__ in_ch_mask, uint8_t *__restrict__ allowed,
                                 int groups, int B, int CD, int K) {
    int64_t total = (int64_t)groups * K;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        int gc = (int)(i / K);
        int j = (int)(i - (int64_t)gc * K);
        allowed[i] = in_ch_mask[gc * B + j / CD] ? 1 : 0;
    }
}

// ---------------------------------------------------------------- scores
__device__ inline float masked(float v, uint8_t keep) { return keep ? v : 0.0f; }

// O_a = sum_j (double)v_aj^2 for each filter a (Section 4, filter-wise set).
// Every wavefront takes one item: R = 4 rows when a row has at most 64 float4
// (one per lane), 2 rows up to 128, else one 1024-weight chunk of a row, whose
// partial sums k_select adds in chunk order.
__device__ inline float4 row_v(const RowLayer &L, const uint8_t *al, const uint8_t *im, int64_t base, int i) {
    float4 x = *reinterpret_cast<const float4 *>(L.W + base + 4 * (int64_t)i);
    float4 y = *reinterpret_cast<const float4 *>(L.U + base + 4 * (int64_t)i);
    float4 v = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
    if (al) {
        uchar4 m = reinterpret_cast<const uchar4 *>(al)[i];
        v.x = masked(v.x, m.x); v.y = masked(v.y, m.y);
        v.z = masked(v.z, m.z); v.w = masked(v.w, m.w);
    } else if (im) {  // the input channel of column j is j / CD
        const uint32_t j = 4u * (uint32_t)i;
        v.x = masked(v.x, im[fdiv(j, L.divCD)]); v.y = masked(v.y, im[fdiv(j + 1, L.divCD)]);
        v.z = masked(v.z, im[fdiv(j + 2, L.divCD)]); v.w = masked(v.w, im[fdiv(j + 3, L.divCD)]);
    }
    return v;
}
__device__ inline const uint8_t *row_inmask(const RowLayer &L, int a) {
    return L.inmask ? L.inmask + (int64_t)(a / L.Ag) * L.B : nullptr;
}
__device__ inline double sq4(float4 v) {
    double acc = (double)v.x * (double)v.x;
    acc += (double)v.y * (double)v.y;
    acc += (double)v.z * (double)v.z;
    acc += (double)v.w * (double)v.w;
    return acc;
}

__global__ __launch_bounds__(kRowThreads) void k_row_scores(RowTab tab) {
    const int li = find_layer(tab.begin, tab.nl, blockIdx.x);
    const RowLayer &L = tab.L[li];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    constexpr int kWaves = kRowThreads / kWave;
    // kRowItems consecutive work items per wavefront, all of their loads issued together
    const int item0 = ((blockIdx.x - tab.begin[li]) * kWaves + wave) * kRowItems;
    if (!L.vec) {  // item = row
        for (int a = item0; a < item0 + kRowItems && a < L.A; ++a) {
            const int64_t base = (int64_t)a * L.K;
            const uint8_t *al = L.allowed ? L.allowed + (int64_t)(a / L.Ag) * L.K : nullptr;
            const uint8_t *im = row_inmask(L, a);
            double acc = 0.0;
            for (int i = lane; i < L.K; i += kWave) {
                float v = L.W[base + i] + L.U[base + i];
                if (al) v = masked(v, al[i]);
                else if (im) v = masked(v, im[fdiv((uint32_t)i, L.divCD)]);
                acc += (double)v * (double)v;
            }
            acc = wave_sum(acc);
            if (lane == 0) L.scores[a] = acc;
        }
        return;
    }
    const int K4 = L.K >> 2;
    float4 v[kRowItems][4];
    if (L.R > 1) {  // item = R short rows; slot u: row a0 + u / (4 / R), float4 lane + 64 * (u % (4 / R))
        const int R = L.R;
#pragma unroll
        for (int q = 0; q < kRowItems; ++q)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int a = (item0 + q) * R + u / (4 / R), i = lane + kWave * (u % (4 / R));
                v[q][u] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (a < L.A && i < K4) {
                    const uint8_t *al = L.allowed ? L.allowed + (int64_t)(a / L.Ag) * L.K : nullptr;
                    v[q][u] = row_v(L, al, row_inmask(L, a), (int64_t)a * L.K, i);
                }
            }
#pragma unroll
        for (int q = 0; q < kRowItems; ++q) {
            const int a0 = (item0 + q) * R;
            if (a0 >= L.A) break;
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int u = 0; u < 4; ++u) acc[u / (4 / R)] += sq4(v[q][u]);
            for (int r = 0; r < R; ++r) {
                const double t = wave_sum(acc[r]);
                if (lane == 0 && a0 + r < L.A) L.scores[a0 + r] = t;
            }
        }
        return;
    }
    // item = (row, chunk of 256 float4): long rows spread over several wavefronts
#pragma unroll
    for (int q = 0; q < kRowItems; ++q) {
        const int item = item0 + q;
        const int a = item / L.nchunk, c = item - a * L.nchunk;
        const uint8_t *al = (L.allowed && a < L.A) ? L.allowed + (int64_t)(a / L.Ag) * L.K : nullptr;
        const uint8_t *im = a < L.A ? row_inmask(L, a) : nullptr;
        const int64_t base = (int64_t)a * L.K;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = c * 4 * kWave + u * kWave + lane;
            v[q][u] = (a < L.A && i < K4) ? row_v(L, al, im, base, i) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
#pragma unroll
    for (int q = 0; q < kRowItems; ++q) {
        const int item = item0 + q;
        const int a = item / L.nchunk, c = item - a * L.nchunk;
        if (a >= L.A) break;
        double acc = 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) acc += sq4(v[q][u]);
        acc = wave_sum(acc);
        if (lane == 0) {
            if (L.nchunk == 1) L.scores[a] = acc;
            else L.rowpart[(int64_t)a * L.nchunk + c] = acc;
        }
    }
}

// partials[band][j] = sum over rows a of the band of (double)v_aj^2
// (column sums; channel and shape scores are finished in k_select).  The four
// wavefronts of a workgroup take 8-row slices of the 32-row band; the slice
// sums are added in slice order.
__global__ __launch_bounds__(kColThreads) void k_col_partials(ColTab tab) {
    constexpr int kLanes = kColThreads / kColSlices;
    __shared__ double red[kColSlices - 1][kLanes * 4];
    const int li = find_layer(tab.begin, tab.nl, blockIdx.x);
    const ColLayer &L = tab.L[li];
    const int lb = blockIdx.x - tab.begin[li];
    const int band = lb / L.ctiles, ct = lb - band * L.ctiles;
    const int lane = threadIdx.x % kLanes, slice = threadIdx.x / kLanes;
    const int a0 = min(L.A, band * kColBand + slice * (kColBand / kColSlices));
    const int a1 = min(L.A, a0 + kColBand / kColSlices);
    const int cw = L.vec ? 4 : 1;  // columns per lane
    const int j = (ct * kLanes + lane) * cw;
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if (j < L.K) {
        if (L.vec) {
            for (int a = a0; a < a1; ++a) {
                const int64_t off = (int64_t)a * L.K + j;
                float4 x = *reinterpret_cast<const float4 *>(L.W + off);
                float4 y = *reinterpret_cast<const float4 *>(L.U + off);
                float v0 = x.x + y.x, v1 = x.y + y.y, v2 = x.z + y.z, v3 = x.w + y.w;
                if (L.allowed) {
                    uchar4 m = *reinterpret_cast<const uchar4 *>(L.allowed + (int64_t)(a / L.Ag) * L.K + j);
                    v0 = masked(v0, m.x); v1 = masked(v1, m.y);
                    v2 = masked(v2, m.z); v3 = masked(v3, m.w);
                }
                s[0] += (double)v0 * (double)v0;
                s[1] += (double)v1 * (double)v1;
                s[2] += (double)v2 * (double)v2;
                s[3] += (double)v3 * (double)v3;
            }
        } else {
            for (int a = a0; a < a1; ++a) {
                const int64_t off = (int64_t)a * L.K + j;
                float v = L.W[off] + L.U[off];
                if (L.allowed) v = masked(v, L.allowed[(int64_t)(a / L.Ag) * L.K + j]);
                s[0] += (double)v * (double)v;
            }
        }
    }
    if (slice > 0)
        for (int c = 0; c < 4; ++c) red[slice - 1][lane * 4 + c] = s[c];
    __syncthreads();
    if (slice == 0 && j < L.K) {
        double *p = L.partials + (int64_t)band * L.K + j;
        for (int c = 0; c < cw; ++c) {
            double t = s[c];
#pragma unroll
            for (int q = 0; q < kColSlices - 1; ++q) t += red[q][lane * 4 + c];
            p[c] = t;
        }
    }
}

// ---------------------------------------------------------------- select
// One workgroup per structured layer.  Keeps exactly k groups: the first k
// of the order (score descending, index ascending), i.e. every group whose
// score exceeds the k-th largest score T plus the lowest-index groups that
// tie with it.  Scores are non-negative binary64, so their bit patterns order
// like unsigned integers: T is found by an MSB-first radix select over the
// 64-bit keys (eight 8-bit digits, one LDS histogram per digit), and the ties
// are ranked by an ordered scan in index order.  Counting is order-free and
// the scans have a fixed order, so the result is reproducible.
__global__ __launch_bounds__(kSelThreads) void k_select(SelTab tab) {
    __shared__ uint64_t skey[SA_MAX_STRUCT_GROUPS];
    __shared__ uint8_t smask[SA_MAX_STRUCT_GROUPS];
    __shared__ uint32_t hist[256];
    __shared__ uint32_t scan_tmp[kSelThreads / kWave + 1];
    __shared__ uint64_t s_prefix;
    __shared__ uint32_t s_need, s_class;

    const SelLayer &L = tab.L[blockIdx.x];
    const int tid = threadIdx.x, lane = tid & 63;
    const int G = L.G;

    // 1. final scores
    for (int g = tid; g < G; g += kSelThreads) {
        double s;
        if (L.kind == SA_FILTER) {
            if (L.rowpart) {  // chunk partials, added in chunk order
                s = 0.0;
                for (int c = 0; c < L.nchunk; ++c) s += L.rowpart[(int64_t)g * L.nchunk + c];
            } else {
                s = L.scores[g];
            }
        } else {
            // shape: over bands; channel: over taps, then bands.  The terms are
            // loaded 16 at a time (every load in flight together) and added in
            // that order; the padding terms past the end add +0 to a sum of
            // squares, which leaves it unchanged.
            const int taps = L.kind == SA_SHAPE ? 1 : L.CD, nb = L.nbands;
            const double *base = L.partials + (L.kind == SA_SHAPE ? g : g * L.CD);
            const int n = taps * nb;
            int t = 0, b = 0;
            s = 0.0;
            for (int i0 = 0; i0 < n; i0 += 16) {
                double v[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    v[q] = i0 + q < n ? base[(int64_t)b * L.K + t] : 0.0;
                    if (++b == nb) {
                        b = 0;
                        ++t;
                    }
                }
#pragma unroll
                for (int q = 0; q < 16; ++q) s += v[q];
            }
        }
        if (L.kind != SA_FILTER || L.rowpart) L.scores[g] = s;
        skey[g] = (uint64_t)__double_as_longlong(s);
        smask[g] = 0;
    }
    __syncthreads();

    // 2. k-th largest key T, and how many of the keys equal to T are kept
    const int per = (G + kSelThreads - 1) / kSelThreads;
    const int g0 = min(G, tid * per), g1 = min(G, g0 + per);
    if (L.k > 0 && L.k < G) {
        uint64_t prefix = 0, pmask = 0;
        uint32_t need = (uint32_t)L.k;  // rank of T among the keys matching prefix
        for (int shift = 56; shift >= 0; shift -= 8) {
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            // the keys of a wavefront that share the first matching key's
            // digit are counted with one atomic (in the leading digits most
            // keys share one bin)
            for (int g0w = tid - lane; g0w < G; g0w += kSelThreads) {
                const int g = g0w + lane;
                const uint64_t key = g < G ? skey[g] : 0;
                const bool in = g < G && (key & pmask) == prefix;
                const uint32_t dig = (uint32_t)(key >> shift) & 255u;
                const unsigned long long vm = __ballot(in);
                if (vm) {
                    const int leader = (int)__builtin_ctzll(vm);
                    const uint32_t d0 = (uint32_t)__shfl((int)dig, leader);
                    const unsigned long long same = __ballot(in && dig == d0);
                    if (lane == leader) atomicAdd(&hist[d0], (uint32_t)__popcll(same));
                    if (in && dig != d0) atomicAdd(&hist[dig], 1u);
                }
            }
            __syncthreads();
            if (tid < kWave) {
                // lane l owns digits 255-4l .. 252-4l (descending)
                uint32_t c[4], tot = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) tot += (c[q] = hist[255 - 4 * lane - q]);
                const uint32_t incl = wave_incl_scan(tot), excl = incl - tot;
                if (excl < need && need <= incl) {
                    uint32_t cum = excl;
                    for (int q = 0; q < 4; ++q) {
                        if (cum + c[q] >= need) {
                            s_prefix = prefix | ((uint64_t)(255 - 4 * lane - q) << shift);
                            s_need = need - cum;
                            s_class = c[q];
                            break;
                        }
                        cum += c[q];
                    }
                }
            }
            __syncthreads();
            prefix = s_prefix;
            need = s_need;
            pmask |= (uint64_t)255 << shift;
            // every key of the class is kept: no finer digit matters (s_* are
            // rewritten only after the next pass's two barriers)
            if (s_class == need) break;
        }
        // keys whose leading digits exceed the class are kept; keys of the class
        // (all equal when every digit was resolved) are kept in index order
        uint32_t ties = 0;
        for (int g = g0; g < g1; ++g) ties += (skey[g] & pmask) == prefix;
        uint32_t total;
        uint32_t rank = block_excl_scan(ties, scan_tmp, &total);
        for (int g = g0; g < g1; ++g) {
            const uint64_t key = skey[g] & pmask;
            uint8_t keep = key > prefix;
            if (key == prefix) keep = rank++ < need;
            smask[g] = keep;
        }
    } else if (L.k == G) {
        for (int g = tid; g < G; g += kSelThreads) smask[g] = 1;
    }
    __syncthreads();

    // 3. mask and ascending kept list (ordered workgroup scan)
    uint32_t kept_local = 0;
    for (int g = g0; g < g1; ++g) kept_local += smask[g];
    uint32_t total;
    uint32_t pos = block_excl_scan(kept_local, scan_tmp, &total);
    for (int g = g0; g < g1; ++g) {
        L.mask[g] = smask[g];
        if (smask[g] && pos < (uint32_t)L.k) L.kept_idx[pos] = g;
        pos += smask[g];
    }

    // 4. per-column keep bytes for the apply pass
    if (L.colkeep) {
        const int64_t total_cols = (int64_t)L.groups * L.K;
        for (int64_t i = tid; i < total_cols; i += kSelThreads) {
            const int gc = (int)(i / L.K);
            const int j = (int)(i - (int64_t)gc * L.K);
            uint8_t sel = 1;
            if (L.kind == SA_SHAPE) sel = smask[j];
            else if (L.kind == SA_CHANNEL) sel = smask[j / L.CD];
            uint8_t al = L.allowed ? L.allowed[i] : 1;
            L.colkeep[i] = (sel && al) ? 1 : 0;
        }
    }
}

// ---------------------------------------------------------------- apply
// Z = v on kept entries, +0 elsewhere; fused: U' = v - Z, G = rho * ((W - Z) + U').
// Flat float4 stream over the layer; entry e sits at row e / K, column e % K.
struct ApplyLayer {
    const float *W;
    float *U;
    float *Z;
    float *G;
    const uint8_t *rowkeep;  // [A] or null
    const uint8_t *colkeep;  // [groups*K] or null
    const uint8_t *inmask;   // [groups*B] or null: column j of conv group gc is kept when
                             // inmask[gc * B + j / CD] is set
    FastDiv divK, divAg, divCD;
    int32_t n, K, B;
    float rho;
};
struct ApplyTab {
    ApplyLayer L[kTab];
    int32_t begin[kTab + 1];
    int32_t nl;
};

constexpr int kApplyThreads = 256;
constexpr int kApplyVec = 4;  // float4 per thread
constexpr int kApplyChunk = kApplyThreads * kApplyVec * 4;

__device__ inline void apply_one(const ApplyLayer &L, float w, float u, uint32_t row, uint32_t col, bool fused,
                                 float &z, float &un, float &g) {
    bool keep = true;
    if (L.rowkeep) keep = L.rowkeep[row] != 0;
    if (keep && L.colkeep) keep = L.colkeep[(int64_t)fdiv(row, L.divAg) * L.K + col] != 0;
    if (keep && L.inmask) keep = L.inmask[(int64_t)fdiv(row, L.divAg) * L.B + fdiv(col, L.divCD)] != 0;
    const float v = w + u;
    z = keep ? v : 0.0f;
    if (fused) {
        un = v - z;
        const float wz = w - z;
        const float s = wz + un;
        g = L.rho * s;
    }
}

__global__ __launch_bounds__(kApplyThreads) void k_apply(ApplyTab tab) {
    const int li = find_layer(tab.begin, tab.nl, blockIdx.x);
    const ApplyLayer &L = tab.L[li];
    const bool fused = L.G != nullptr;
    const int64_t c0 = (int64_t)(blockIdx.x - tab.begin[li]) * kApplyChunk;
    float4 xw[kApplyVec], xu[kApplyVec];
#pragma unroll
    for (int q = 0; q < kApplyVec; ++q) {
        const int64_t e = c0 + ((int64_t)q * kApplyThreads + threadIdx.x) * 4;
        if (e + 4 <= L.n) {
            xw[q] = *reinterpret_cast<const float4 *>(L.W + e);
            xu[q] = *reinterpret_cast<const float4 *>(L.U + e);
        }
    }
#pragma unroll
    for (int q = 0; q < kApplyVec; ++q) {
        const int64_t e = c0 + ((int64_t)q * kApplyThreads + threadIdx.x) * 4;
        if (e >= L.n) continue;
        if (e + 4 <= L.n) {
            uint32_t row = fdiv((uint32_t)e, L.divK);
            uint32_t col = (uint32_t)e - row * (uint32_t)L.K;
            float w[4] = {xw[q].x, xw[q].y, xw[q].z, xw[q].w};
            float u[4] = {xu[q].x, xu[q].y, xu[q].z, xu[q].w};
            float z[4], un[4], g[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                apply_one(L, w[i], u[i], row, col, fused, z[i], un[i], g[i]);
                if (++col == (uint32_t)L.K) {
                    col = 0;
                    ++row;
                }
            }
            // non-temporal stores: the outputs stream past the caches, which
            // keep W and U (read by the score pass just before) for the loads
            // above (measured 5% faster on the ResNet-50 step, 9% on 1 GB)
            nt_store4(L.Z + e, z);
            if (fused) {
                nt_store4(L.U + e, un);
                nt_store4(L.G + e, g);
            }
        } else {
            for (int64_t f = e; f < L.n; ++f) {
                uint32_t row = fdiv((uint32_t)f, L.divK);
                uint32_t col = (uint32_t)f - row * (uint32_t)L.K;
                float z, un = 0.f, g = 0.f;
                apply_one(L, L.W[f], L.U[f], row, col, fused, z, un, g);
                L.Z[f] = z;
                if (fused) {
                    L.U[f] = un;
                    L.G[f] = g;
                }
            }
        }
    }
}

// ---------------------------------------------------------------- element-wise
// Every element-wise layer of a dependency level goes through one launch per
// phase: zeroed histograms, three digit histograms of |v|, the counts, the
// apply pass.  Small layers are launch latency: with a launch of its own per
// layer and phase and a one-wavefront kernel between the passes AlexNet's five
// layers (2.3 M weights) took 50 launches and 240 us; now 6 launches and 44 us.
struct ElemState {
    uint32_t prefix;  // digits of T found so far; after the last pass, T itself
    uint32_t kk;      // rank of T among keys matching the prefix
};

struct ElemLayer {
    const float *W;
    float *U;
    float *Z;
    float *G;
    uint8_t *mask;
    int32_t *kept_idx;
    double *scores;         // [n] keys as |v| in binary64, or null
    const uint8_t *inmask;  // [groups*B] input-channel support, or null
    uint32_t *hist;         // [3][2048]
    ElemState *state;       // [3]: after the first, second and third digit
    uint2 *counts;          // keys above T and equal to T of each block's range
    FastDiv divK, divAg, divCD;
    int32_t n, K, B, k;
    int32_t sub, hsub;  // chunks of kElemChunk entries per block, of kHistChunk per histogram block
    float rho;
};
struct ElemTab {
    ElemLayer L[kElemTab];
    int32_t begin[kElemTab + 1];   // first block of each layer
    int32_t hbegin[kElemTab + 1];  // and of the histogram passes
    int32_t nl;
};

static_assert(sizeof(RowTab) < 8192 && sizeof(ColTab) < 8192 && sizeof(SelTab) < 8192 &&
                  sizeof(DualTab) < 8192 && sizeof(ApplyTab) < 8192 && sizeof(SgdTab) < 8192 && sizeof(ElemTab) < 8192,
              "layer tables must fit the kernel-argument segment");

// Is entry e inside the input-channel support?
__device__ inline bool elem_allowed(uint32_t e, const ElemLayer &a) {
    if (!a.inmask) return true;
    const uint32_t row = fdiv(e, a.divK);
    return a.inmask[fdiv(row, a.divAg) * (uint32_t)a.B + fdiv(e - row * (uint32_t)a.K, a.divCD)] != 0;
}

// Key of entry e: |v| as binary32 bits (sign cleared); 0 outside the support.
__device__ inline uint32_t elem_key(float v, uint32_t e, const ElemLayer &a) {
    const uint32_t key = __float_as_uint(v) & 0x7fffffffu;
    return elem_allowed(e, a) ? key : 0u;
}

__device__ inline void elem_load8(const ElemLayer &a, int64_t e0, float *w, float *v) {
    if (e0 + 8 <= a.n) {  // e0 is a multiple of 8, W and U are 16-byte aligned
        float4 w0 = *reinterpret_cast<const float4 *>(a.W + e0);
        float4 w1 = *reinterpret_cast<const float4 *>(a.W + e0 + 4);
        float4 u0 = *reinterpret_cast<const float4 *>(a.U + e0);
        float4 u1 = *reinterpret_cast<const float4 *>(a.U + e0 + 4);
        w[0] = w0.x; w[1] = w0.y; w[2] = w0.z; w[3] = w0.w;
        w[4] = w1.x; w[5] = w1.y; w[6] = w1.z; w[7] = w1.w;
        v[0] = w0.x + u0.x; v[1] = w0.y + u0.y; v[2] = w0.z + u0.z; v[3] = w0.w + u0.w;
        v[4] = w1.x + u1.x; v[5] = w1.y + u1.y; v[6] = w1.z + u1.z; v[7] = w1.w + u1.w;
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            int64_t e = e0 + q;
            if (e < a.n) {
                w[q] = a.W[e];
                v[q] = w[q] + a.U[e];
            } else {
                w[q] = 0.f;
                v[q] = 0.f;
            }
        }
    }
}

__global__ __launch_bounds__(kHistThreads) void k_elem_init(ElemTab tab) {
    uint32_t *h = tab.L[blockIdx.x].hist;
    for (int i = threadIdx.x; i < 3 * 2048; i += kHistThreads) h[i] = 0;
}

// The digit of pass `pass` that holds the kk-th largest key, and the rank
// within it: every workgroup works it out for itself from the finished
// histogram (2048 or 512 bins, a few per thread), which spares a launch
// between the passes.  `tmp` and `out`: LDS of the workgroup.
template <int kThreads, int kBits>
__device__ inline ElemState elem_find(const ElemLayer &a, int pass, ElemState s, uint32_t *tmp, ElemState *out) {
    constexpr int kPer = (1 << kBits) / kThreads;
    const int top = (1 << kBits) - 1 - (int)threadIdx.x * kPer;  // descending
    const uint32_t *gh = a.hist + pass * 2048 + top;
    uint32_t c[kPer], sum = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) sum += (c[q] = gh[-q]);
    uint32_t total;
    uint32_t above = block_excl_scan(sum, tmp, &total);
    if (above < s.kk && s.kk <= above + sum) {  // exactly one thread
        int q = 0;
#pragma unroll
        for (int i = 0; i + 1 < kPer; ++i)
            if (q == i && above + c[i] < s.kk) {
                above += c[i];
                q = i + 1;
            }
        *out = ElemState{(s.prefix << kBits) | (uint32_t)(top - q), s.kk - above};
    }
    __syncthreads();
    return *out;
}

// Histogram of one digit of the keys that match the digits found so far.
// Digits: pass 0 = bits 30..20, pass 1 = bits 19..9, pass 2 = bits 8..0.
// Adding the workgroups' histograms up in memory bounds the pass (the reads
// alone take 3 us of AlexNet's 2.3 M weights), so a workgroup is large: 7.9,
// 9.2 and 6.9 us with 1024 threads, 8.4, 12 and 7.4 with 512, 11.9, 14 and 9.8
// with 256.
__global__ __launch_bounds__(kHistThreads) void k_elem_hist(ElemTab tab, int pass) {
    __shared__ uint32_t h[2048];
    __shared__ uint32_t tmp[kHistThreads / kWave + 1];
    __shared__ ElemState found;
    const int li = find_layer(tab.hbegin, tab.nl, blockIdx.x);
    const ElemLayer &a = tab.L[li];
    if (a.k == 0) return;
    const int blk = blockIdx.x - tab.hbegin[li];
    for (int i = threadIdx.x; i < 2048; i += kHistThreads) h[i] = 0;
    const int64_t first = (int64_t)blk * a.hsub * kHistChunk + (int64_t)threadIdx.x * kElemPerThread;
    float w[8], v[8];
    elem_load8(a, first, w, v);  // in flight while the digit of the pass before is found
    ElemState s{0u, (uint32_t)a.k};
    if (pass > 0) {
        if (pass > 1) s = a.state[pass - 2];
        s = elem_find<kHistThreads, 11>(a, pass - 1, s, tmp, &found);
        if (blk == 0 && threadIdx.x == 0) a.state[pass - 1] = s;
    } else {
        __syncthreads();
    }
    const int dshift = pass == 0 ? 20 : (pass == 1 ? 9 : 0);
    const uint32_t dmask = pass == 2 ? 0x1ffu : 0x7ffu;
    const int mshift = pass == 0 ? 31 : (pass == 1 ? 20 : 9);
    for (int c = 0; c < a.hsub; ++c) {
        const int64_t e0 = first + (int64_t)c * kHistChunk;
        if (c > 0) elem_load8(a, e0, w, v);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (e0 + q >= a.n) break;
            const uint32_t key = elem_key(v[q], (uint32_t)(e0 + q), a);
            if (pass == 0 || (key >> mshift) == s.prefix) atomicAdd(&h[(key >> dshift) & dmask], 1u);
        }
    }
    __syncthreads();
    uint32_t *gh = a.hist + pass * 2048;
    for (int i = threadIdx.x; i < 2048; i += kHistThreads)
        if (h[i]) atomicAdd(&gh[i], h[i]);
}

// Per-block counts of keys above T and equal to T.
__global__ __launch_bounds__(kElemThreads) void k_elem_count(ElemTab tab) {
    __shared__ uint32_t red[2][kElemThreads / kWave];
    __shared__ uint32_t tmp[kElemThreads / kWave + 1];
    __shared__ ElemState found;
    const int li = find_layer(tab.begin, tab.nl, blockIdx.x);
    const ElemLayer &a = tab.L[li];
    const int blk = blockIdx.x - tab.begin[li];
    const int64_t first = (int64_t)blk * a.sub * kElemChunk + (int64_t)threadIdx.x * kElemPerThread;
    float w[8], v[8];
    elem_load8(a, first, w, v);
    ElemState s{0x80000000u, 0u};  // k = 0: T above every key
    if (a.k > 0) s = elem_find<kElemThreads, 9>(a, 2, a.state[1], tmp, &found);
    if (blk == 0 && threadIdx.x == 0) a.state[2] = s;
    uint32_t gt = 0, eq = 0;
    for (int c = 0; c < a.sub; ++c) {
        const int64_t e0 = first + (int64_t)c * kElemChunk;
        if (c > 0) elem_load8(a, e0, w, v);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (e0 + q >= a.n) break;
            const uint32_t key = elem_key(v[q], (uint32_t)(e0 + q), a);
            gt += key > s.prefix;
            eq += key == s.prefix;
        }
    }
    gt = wave_sum_u32(gt);
    eq = wave_sum_u32(eq);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wave] = gt;
        red[1][wave] = eq;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t g = 0, e = 0;
        for (int i = 0; i < kElemThreads / kWave; ++i) {
            g += red[0][i];
            e += red[1][i];
        }
        a.counts[blk] = make_uint2(g, e);
    }
}

// Mask, ascending kept_idx, Z (+ fused U', G) for the non-structured set.  The
// entries kept before a position are the keys above T before it and the first
// `need` keys equal to T; each block adds up the counts of the blocks before it
// (at most kElemMaxBlocks).  Bound by its 16 to 21 bytes an entry; workgroups of
// 256 threads: 12.5 us of AlexNet's 2.3 M weights, 512 take 16.5 and 1024 18.5.
__global__ __launch_bounds__(kElemThreads) void k_elem_apply(ElemTab tab) {
    __shared__ uint32_t tmp[kElemThreads / kWave + 1];
    __shared__ uint32_t red[2][kElemThreads / kWave];
    const int li = find_layer(tab.begin, tab.nl, blockIdx.x);
    const ElemLayer &a = tab.L[li];
    const int blk = blockIdx.x - tab.begin[li];
    const int wave = threadIdx.x >> 6;
    const int64_t first = (int64_t)blk * a.sub * kElemChunk + (int64_t)threadIdx.x * kElemPerThread;
    float w[8], v[8];
    elem_load8(a, first, w, v);
    const uint32_t T = a.state[2].prefix;
    const uint32_t need = a.state[2].kk;  // keys equal to T that are kept (0 when k = 0)
    uint32_t gt_before = 0, eq_before = 0;
    for (int c = threadIdx.x; c < blk; c += kElemThreads) {
        const uint2 t = a.counts[c];
        gt_before += t.x;
        eq_before += t.y;
    }
    gt_before = wave_sum_u32(gt_before);
    eq_before = wave_sum_u32(eq_before);
    if ((threadIdx.x & 63) == 0) {
        red[0][wave] = gt_before;
        red[1][wave] = eq_before;
    }
    __syncthreads();
    gt_before = eq_before = 0;
    for (int i = 0; i < kElemThreads / kWave; ++i) {
        gt_before += red[0][i];
        eq_before += red[1][i];
    }
    const bool fused = a.G != nullptr;
    const bool mvec = ((uintptr_t)a.mask & 7) == 0;
    for (int c = 0; c < a.sub; ++c) {
        const int64_t e0 = first + (int64_t)c * kElemChunk;
        if (c > 0) elem_load8(a, e0, w, v);
        uint32_t key[8], cnt = 0;  // cnt: keys above T, and equal to T in the upper half
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            key[q] = (e0 + q < a.n) ? elem_key(v[q], (uint32_t)(e0 + q), a) : 0u;
            if (e0 + q < a.n) cnt += key[q] > T ? 1u : (key[q] == T ? 0x10000u : 0u);
        }
        uint32_t total;  // at most kElemChunk of either kind: no carry between the halves
        const uint32_t before = block_excl_scan(cnt, tmp, &total);
        uint32_t eq_rank = eq_before + (before >> 16);
        uint32_t pos = gt_before + (before & 0xffffu) + min(eq_rank, need);
        gt_before += total & 0xffffu;
        eq_before += total >> 16;
        float z[8], un[8], g[8];
        uint32_t bits = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t e = e0 + q;
            bool keep = false;
            if (e < a.n && a.k > 0) keep = key[q] > T || (key[q] == T && eq_rank++ < need);
            // a kept entry outside the support (score 0) still projects to 0
            z[q] = (keep && elem_allowed((uint32_t)e, a)) ? v[q] : 0.0f;
            un[q] = v[q] - z[q];
            const float wz = w[q] - z[q];
            const float sum = wz + un[q];
            g[q] = a.rho * sum;
            bits |= keep ? 1u << q : 0u;
            if (keep && pos < (uint32_t)a.k) a.kept_idx[pos] = (int32_t)e;
            pos += keep ? 1u : 0u;
            if (a.scores && e < a.n) a.scores[e] = (double)__uint_as_float(key[q]);
        }
        if (e0 + 8 <= a.n) {
            nt_store4(a.Z + e0, z);
            nt_store4(a.Z + e0 + 4, z + 4);
            if (fused) {
                nt_store4(a.U + e0, un);
                nt_store4(a.U + e0 + 4, un + 4);
                nt_store4(a.G + e0, g);
                nt_store4(a.G + e0 + 4, g + 4);
            }
            // bit q of a nibble to byte q
            const uint32_t lo = ((bits & 15u) * 0x00204081u) & 0x01010101u;
            const uint32_t hi = ((bits >> 4) * 0x00204081u) & 0x01010101u;
            if (mvec) {
                *reinterpret_cast<uint2 *>(a.mask + e0) = make_uint2(lo, hi);
            } else {
#pragma unroll
                for (int q = 0; q < 8; ++q) a.mask[e0 + q] = (uint8_t)((bits >> q) & 1u);
            }
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int64_t e = e0 + q;
                if (e >= a.n) break;
                a.Z[e] = z[q];
                a.mask[e] = (uint8_t)((bits >> q) & 1u);
                if (fused) {
                    a.U[e] = un[q];
                    a.G[e] = g[q];
                }
            }
        }
    }
}

// ---------------------------------------------------------------- dual
constexpr int kDualThreads = 256;
constexpr int kDualVecPerThread = 4;  // float4 per thread per workgroup pass
constexpr int kDualChunk = kDualThreads * kDualVecPerThread * 4;

// U <- (U + W) - Z;  G = rho * ((W - Z) + U)   (U new, or unchanged if !update)
__global__ __launch_bounds__(kDualThreads) void k_dual(DualTab tab) {
    const int li = find_layer(tab.begin, tab.nl, blockIdx.x);
    const DualLayer &L = tab.L[li];
    const int64_t c0 = (int64_t)(blockIdx.x - tab.begin[li]) * kDualChunk;
    const int n4 = L.n >> 2;
    // every load of the thread issued before any store; U and G are written
    // with the non-temporal hint (streamed past the caches: measured 72.7 ->
    // 56.9 us for the 23.45 M-weight ResNet-50 gradient pass)
    float4 w[kDualVecPerThread], z[kDualVecPerThread], uu[kDualVecPerThread];
#pragma unroll
    for (int u = 0; u < kDualVecPerThread; ++u) {
        const int64_t i = (c0 >> 2) + (int64_t)u * kDualThreads + threadIdx.x;
        if (i < n4) {
            w[u] = reinterpret_cast<const float4 *>(L.W)[i];
            z[u] = reinterpret_cast<const float4 *>(L.Z)[i];
            uu[u] = reinterpret_cast<const float4 *>(L.U)[i];
        }
    }
#pragma unroll
    for (int u = 0; u < kDualVecPerThread; ++u) {
        const int64_t i = (c0 >> 2) + (int64_t)u * kDualThreads + threadIdx.x;
        if (i < n4) {
            float wv[4] = {w[u].x, w[u].y, w[u].z, w[u].w}, zv[4] = {z[u].x, z[u].y, z[u].z, z[u].w};
            float uv[4] = {uu[u].x, uu[u].y, uu[u].z, uu[u].w}, gv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (L.update) {
                    float s = uv[e] + wv[e];
                    uv[e] = s - zv[e];
                }
                float wz = wv[e] - zv[e];
                float t = wz + uv[e];
                gv[e] = L.rho * t;
            }
            if (L.update) nt_store4(reinterpret_cast<float *>(L.U) + 4 * i, uv);
            if (L.G) nt_store4(reinterpret_cast<float *>(L.G) + 4 * i, gv);
        }
    }
    // scalar tail (n % 4 entries), handled by the layer's first workgroup
    if (blockIdx.x == tab.begin[li] && threadIdx.x < (L.n & 3)) {
        const int64_t e = (int64_t)n4 * 4 + threadIdx.x;
        float u = L.U[e];
        if (L.update) {
            float s = u + L.W[e];
            u = s - L.Z[e];
            L.U[e] = u;
        }
        if (L.G) {
            float wz = L.W[e] - L.Z[e];
            float t = wz + u;
            L.G[e] = L.rho * t;
        }
    }
}

// ---------------------------------------------------------------- SGD step
constexpr int kSgdThreads = 256;
constexpr int kSgdVecPerThread = 4;
constexpr int kSgdChunk = kSgdThreads * kSgdVecPerThread * 4;

__device__ inline bool sgd_keep(const SgdLayer &L, uint32_t e) {
    if (!L.mask) return true;
    uint32_t g = e;
    if (L.kind != SA_ELEMENT) {
        const uint32_t a = fdiv(e, L.divK);
        const uint32_t j = e - a * L.divK.d;  // column (b*C + c)*D + d
        g = L.kind == SA_FILTER ? a : L.kind == SA_CHANNEL ? fdiv(j, L.divCD) : j;
    }
    return L.mask[g] != 0;
}

// t = Gf + rho * ((W - Z) + U) (or Gf);  W <- keep ? W - lr * t : +0
__device__ inline float sgd_one(const SgdLayer &L, float w, float gf, float z, float u, bool keep) {
    float t = gf;
    if (L.Z) {
        const float d = w - z;
        const float sum = d + u;
        const float r = L.rho * sum;
        t = gf + r;
    }
    const float q = L.lr * t;
    return keep ? w - q : 0.0f;
}

__global__ __launch_bounds__(kSgdThreads) void k_sgd(SgdTab tab) {
    const int li = find_layer(tab.begin, tab.nl, blockIdx.x);
    const SgdLayer &L = tab.L[li];
    const int64_t c0 = (int64_t)(blockIdx.x - tab.begin[li]) * kSgdChunk;
    const int n4 = L.n >> 2;
#pragma unroll
    for (int v = 0; v < kSgdVecPerThread; ++v) {
        const int64_t i = (c0 >> 2) + (int64_t)v * kSgdThreads + threadIdx.x;
        if (i < n4) {
            const float4 w = reinterpret_cast<const float4 *>(L.W)[i];
            const float4 g = reinterpret_cast<const float4 *>(L.Gf)[i];
            float4 z = make_float4(0.f, 0.f, 0.f, 0.f), u = z;
            if (L.Z) {
                z = reinterpret_cast<const float4 *>(L.Z)[i];
                u = reinterpret_cast<const float4 *>(L.U)[i];
            }
            const uint32_t e = (uint32_t)i * 4u;
            float4 o;
            o.x = sgd_one(L, w.x, g.x, z.x, u.x, sgd_keep(L, e));
            o.y = sgd_one(L, w.y, g.y, z.y, u.y, sgd_keep(L, e + 1));
            o.z = sgd_one(L, w.z, g.z, z.z, u.z, sgd_keep(L, e + 2));
            o.w = sgd_one(L, w.w, g.w, z.w, u.w, sgd_keep(L, e + 3));
            reinterpret_cast<float4 *>(L.W)[i] = o;
        }
    }
    // scalar tail (n % 4 entries), handled by the layer's first workgroup
    if (blockIdx.x == tab.begin[li] && threadIdx.x < (L.n & 3)) {
        const uint32_t e = (uint32_t)n4 * 4u + threadIdx.x;
        const float z = L.Z ? L.Z[e] : 0.f, u = L.Z ? L.U[e] : 0.f;
        L.W[e] = sgd_one(L, L.W[e], L.Gf[e], z, u, sgd_keep(L, e));
    }
}

// ---------------------------------------------------------------- host planning
struct LayerPlan {
    int64_t G;
    int K, CD, Ag, R, rchunks, ritems, nbands, ctiles, vec, nblk, sub, hblk, hsub;
    size_t off_scores, off_rowpart, off_partials, off_allowed, off_colkeep, off_elem;
    size_t end;
};

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

void plan_layer(const sa_project_desc &d, size_t start, LayerPlan &p) {
    p.G = n_groups(d);
    p.K = (int)(d.B * d.C * d.D);
    p.CD = (int)(d.C * d.D);
    p.Ag = (int)(d.A / d.groups);
    p.vec = (p.K % 4 == 0) ? 1 : 0;
    // filter scores: work items of one wavefront each
    const int K4 = p.K / 4;
    p.R = !p.vec ? 1 : (K4 <= kWave ? 4 : (K4 <= 2 * kWave ? 2 : 1));
    p.rchunks = (p.vec && p.R == 1) ? (K4 + 4 * kWave - 1) / (4 * kWave) : 1;
    p.ritems = !p.vec ? (int)d.A : (p.R > 1 ? (int)((d.A + p.R - 1) / p.R) : (int)d.A * p.rchunks);
    p.nbands = (int)((d.A + kColBand - 1) / kColBand);
    const int cols_per_block = (kColThreads / kColSlices) * (p.vec ? 4 : 1);
    p.ctiles = (p.K + cols_per_block - 1) / cols_per_block;
    const int64_t n = d.A * d.B * d.C * d.D;
    const int64_t chunks = (n + kElemChunk - 1) / kElemChunk;
    p.sub = (int)((chunks + kElemMaxBlocks - 1) / kElemMaxBlocks);
    p.nblk = (int)((chunks + p.sub - 1) / p.sub);
    const int64_t hchunks = (n + kHistChunk - 1) / kHistChunk;
    p.hsub = (int)((hchunks + kElemMaxBlocks - 1) / kElemMaxBlocks);
    p.hblk = (int)((hchunks + p.hsub - 1) / p.hsub);
    size_t off = align256(start);
    p.off_scores = p.off_rowpart = p.off_partials = p.off_allowed = p.off_colkeep = p.off_elem = SIZE_MAX;
    if (d.kind != SA_ELEMENT && !d.scores) {
        p.off_scores = off;
        off = align256(off + sizeof(double) * p.G);
    }
    if (d.kind == SA_FILTER && p.rchunks > 1) {
        p.off_rowpart = off;
        off = align256(off + sizeof(double) * (size_t)d.A * p.rchunks);
    }
    if (d.kind == SA_CHANNEL || d.kind == SA_SHAPE) {
        p.off_partials = off;
        off = align256(off + sizeof(double) * (size_t)p.nbands * p.K);
    }
    if (d.in_ch_mask && d.kind != SA_FILTER) {
        p.off_allowed = off;
        off = align256(off + (size_t)d.groups * p.K);
    }
    if (d.kind == SA_CHANNEL || d.kind == SA_SHAPE) {
        p.off_colkeep = off;
        off = align256(off + (size_t)d.groups * p.K);
    }
    if (d.kind == SA_ELEMENT) {
        p.off_elem = off;
        // 16 bytes per chunk: the counts need 8 per block; the size callers
        // were told, and with it what the held scratch takes, stays the same
        off = align256(off + sizeof(uint32_t) * 3 * 2048 + 16 + 256 + 16 * (size_t)chunks);
    }
    p.end = off;
}

template <typename T>
T *ws_at(void *ws, size_t off) {
    return reinterpret_cast<T *>(static_cast<char *>(ws) + off);
}

int launch_check(const char *what) { return check_hip(hipGetLastError(), what); }

// Bytes [lo, hi) of a buffer; empty for a null pointer.
struct Span {
    uintptr_t lo, hi;
};
Span span(const void *p, int64_t bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p);
    return p ? Span{a, a + (uintptr_t)bytes} : Span{0, 0};
}
template <size_t M, size_t N>
bool meet(const std::array<Span, M> &a, const std::array<Span, N> &b) {
    for (const Span &p : a)
        for (const Span &q : b)
            if (p.lo < q.hi && q.lo < p.hi) return true;
    return false;
}

int64_t entries(const sa_project_desc &d) { return d.A * d.B * d.C * d.D; }

// What the projection of a layer writes, and what it reads besides its support.
std::array<Span, 6> written(const sa_project_desc &d) {
    const int64_t n = entries(d), g = n_groups(d);
    return {span(d.Z, n * 4), span(d.mask, g),    span(d.kept_idx, d.k * 4), span(d.scores, g * 8),
            span(d.G, n * 4), span(d.G ? d.U : nullptr, n * 4)};
}
std::array<Span, 2> read(const sa_project_desc &d) {
    return {span(d.W, entries(d) * 4), span(d.U, entries(d) * 4)};
}

}  // namespace
}  // namespace sa

using namespace sa;

extern "C" size_t structadmm_project_workspace(const sa_project_desc *layers, int n_layers) {
    if (!layers || n_layers <= 0) return 0;
    size_t off = 0;
    for (int i = 0; i < n_layers; ++i) {
        if (validate_project(layers[i], i) != SA_OK) {
            clear_error();
            return 0;
        }
        LayerPlan p;
        plan_layer(layers[i], off, p);
        off = p.end;
    }
    return off;
}

namespace sa {
namespace {

// Scratch of structadmm_project_noalloc: one copy per GPU, in the code
// object's device memory, held until the process ends.  Host code never uses
// the symbol itself as an address: the device address of each GPU's copy
// comes from hipGetSymbolAddress with that GPU current.
__device__ __align__(256) uint8_t scratch[SA_PROJECT_NOALLOC_BYTES];

constexpr int kMaxDevices = 64;

// Device address of the current GPU's scratch (nullptr and an error set on failure).
void *noalloc_scratch() {
    static std::mutex mu;
    static void *ptr[kMaxDevices] = {};
    int dev = 0;
    if (check_hip(hipGetDevice(&dev), "project_noalloc: current device")) return nullptr;
    if (dev < 0 || dev >= kMaxDevices) {
        fail(SA_E_UNSUPPORTED, "project_noalloc: device index %d beyond %d", dev, kMaxDevices);
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        if (check_hip(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "project_noalloc: scratch address")) return nullptr;
        ptr[dev] = p;
    }
    return ptr[dev];
}

int project_impl(const sa_project_desc *layers, int n_layers, void *ws, size_t ws_bytes, hipStream_t stream);

}  // namespace
}  // namespace sa

extern "C" int structadmm_project(const sa_project_desc *layers, int n_layers, void *ws,
                                  size_t ws_bytes, hipStream_t stream) {
    clear_error();
    return project_impl(layers, n_layers, ws, ws_bytes, stream);
}

extern "C" int structadmm_project_noalloc(const sa_project_desc *layers, int n_layers, hipStream_t stream) {
    clear_error();
    if (!layers || n_layers <= 0) return fail(SA_E_ARG, "project: layers must be a non-empty array");
    size_t need = 0;
    for (int i = 0; i < n_layers; ++i) {
        if (int rc = validate_project(layers[i], i)) return rc;
        LayerPlan p;
        plan_layer(layers[i], need, p);
        need = p.end;
    }
    if (need > (size_t)SA_PROJECT_NOALLOC_BYTES)
        return fail(SA_E_WORKSPACE, "project_noalloc: these layers need %zu bytes of scratch, more than the %zu "
                    "the library holds (use structadmm_project with a workspace)", need,
                    (size_t)SA_PROJECT_NOALLOC_BYTES);
    void *ws = need > 0 ? noalloc_scratch() : nullptr;
    if (need > 0 && !ws) return SA_E_HIP;
    return project_impl(layers, n_layers, ws, SA_PROJECT_NOALLOC_BYTES, stream);
}

namespace sa {
namespace {

int project_impl(const sa_project_desc *layers, int n_layers, void *ws, size_t ws_bytes, hipStream_t stream) {
    if (!layers || n_layers <= 0) return fail(SA_E_ARG, "project: layers must be a non-empty array");
    std::vector<LayerPlan> plan(n_layers);
    size_t off = 0;
    for (int i = 0; i < n_layers; ++i) {
        int rc = validate_project(layers[i], i);
        if (rc) return rc;
        plan_layer(layers[i], off, plan[i]);
        off = plan[i].end;
    }
    if (off > 0) {
        if (!ws) return fail(SA_E_WORKSPACE, "project: workspace of %zu bytes required", off);
        if (ws_bytes < off)
            return fail(SA_E_WORKSPACE, "project: workspace %zu bytes < required %zu", ws_bytes, off);
        if (!aligned(ws, 256)) return fail(SA_E_ALIGN, "project: workspace must be 256-byte aligned");
    }
    // dependency levels: a layer whose in_ch_mask is an earlier layer's mask runs after it
    std::vector<int> level(n_layers, 0);
    int max_level = 0;
    for (int i = 0; i < n_layers; ++i) {
        for (int j = 0; j < i; ++j)
            if (layers[i].in_ch_mask && (const void *)layers[i].in_ch_mask == (const void *)layers[j].mask)
                level[i] = std::max(level[i], level[j] + 1);
        max_level = std::max(max_level, level[i]);
    }

    // May layer ids[m] share launches with layers ids[0..m)?  Layers of a level
    // run in the order given where one writes what another reads or writes.
    auto apart = [](const sa_project_desc *l, const int *ids, int m) {
        const sa_project_desc &b = l[ids[m]];
        for (int j = 0; j < m; ++j) {
            const sa_project_desc &a = l[ids[j]];
            if (meet(written(a), written(b)) || meet(written(a), read(b)) || meet(written(b), read(a))) return false;
        }
        return true;
    };

    auto fill_row = [&](int i, RowLayer &R) {
        const sa_project_desc &d = layers[i];
        const LayerPlan &p = plan[i];
        R.W = d.W;
        R.U = d.U;
        // filter sets read their support straight from the input-channel mask;
        // the other sets use its per-column expansion
        R.allowed = d.in_ch_mask && d.kind != SA_FILTER ? ws_at<uint8_t>(ws, p.off_allowed) : nullptr;
        R.inmask = d.kind == SA_FILTER ? d.in_ch_mask : nullptr;
        R.B = (int)d.B;
        R.divCD = make_fastdiv((uint32_t)p.CD);
        R.scores = d.scores ? d.scores : (p.off_scores != SIZE_MAX ? ws_at<double>(ws, p.off_scores) : nullptr);
        R.A = (int)d.A;
        R.K = p.K;
        R.Ag = p.Ag;
        R.R = p.R;
        R.nchunk = p.rchunks;
        R.rowpart = p.off_rowpart != SIZE_MAX ? ws_at<double>(ws, p.off_rowpart) : nullptr;
        R.vec = p.vec;
        R.rho = d.rho;
    };

    for (int lv = 0; lv <= max_level; ++lv) {
        std::vector<int> ids;
        for (int i = 0; i < n_layers; ++i)
            if (level[i] == lv) ids.push_back(i);

        // Allowed bytes for layers with a channel support (filter sets read the
        // mask itself).  An element-wise layer reads the mask itself too, unless
        // a layer of this level writes over it (its own mask, one that a later
        // layer selects, a place inside another buffer): then it reads a copy
        // from before the level, one byte per channel.
        std::vector<char> held(n_layers, 0);
        for (int i : ids) {
            const sa_project_desc &d = layers[i];
            if (!d.in_ch_mask || d.kind == SA_FILTER) continue;
            const LayerPlan &p = plan[i];
            int K = p.K, CD = p.CD;
            if (d.kind == SA_ELEMENT) {
                const std::array<Span, 1> sup = {span(d.in_ch_mask, (int64_t)d.groups * d.B)};
                for (int j : ids) held[i] = held[i] || meet(sup, written(layers[j]));
                if (!held[i]) continue;
                K = (int)d.B;
                CD = 1;
            }
            int64_t total = (int64_t)d.groups * K;
            int blocks = (int)std::min<int64_t>(1024, (total + 255) / 256);
            hipLaunchKernelGGL(k_expand_allowed, dim3(blocks), dim3(256), 0, stream, d.in_ch_mask,
                               ws_at<uint8_t>(ws, p.off_allowed), d.groups, (int)d.B, CD, K);
            if (int rc = launch_check("k_expand_allowed")) return rc;
        }


        // filter scores
        {
            std::vector<int> f;
            for (int i : ids)
                if (layers[i].kind == SA_FILTER) f.push_back(i);
            for (size_t s = 0; s < f.size(); s += kTab) {
                RowTab tab;
                memset(&tab, 0, sizeof tab);
                int blocks = 0;
                tab.nl = (int)std::min<size_t>(kTab, f.size() - s);
                for (int t = 0; t < tab.nl; ++t) {
                    fill_row(f[s + t], tab.L[t]);
                    tab.begin[t] = blocks;
                    blocks += (plan[f[s + t]].ritems + kRowItems * (kRowThreads / kWave) - 1) /
                              (kRowItems * (kRowThreads / kWave));
                }
                tab.begin[tab.nl] = blocks;
                hipLaunchKernelGGL(k_row_scores, dim3(blocks), dim3(kRowThreads), 0, stream, tab);
                if (int rc = launch_check("k_row_scores")) return rc;
            }
        }
        // channel / shape column partials
        {
            std::vector<int> c;
            for (int i : ids)
                if (layers[i].kind == SA_CHANNEL || layers[i].kind == SA_SHAPE) c.push_back(i);
            for (size_t s = 0; s < c.size(); s += kTab) {
                ColTab tab;
                memset(&tab, 0, sizeof tab);
                int blocks = 0;
                tab.nl = (int)std::min<size_t>(kTab, c.size() - s);
                for (int t = 0; t < tab.nl; ++t) {
                    const sa_project_desc &d = layers[c[s + t]];
                    const LayerPlan &p = plan[c[s + t]];
                    ColLayer &L = tab.L[t];
                    L.W = d.W;
                    L.U = d.U;
                    L.allowed = d.in_ch_mask ? ws_at<uint8_t>(ws, p.off_allowed) : nullptr;
                    L.partials = ws_at<double>(ws, p.off_partials);
                    L.A = (int)d.A;
                    L.K = p.K;
                    L.Ag = p.Ag;
                    L.nbands = p.nbands;
                    L.ctiles = p.ctiles;
                    L.vec = p.vec;
                    tab.begin[t] = blocks;
                    blocks += p.nbands * p.ctiles;
                }
                tab.begin[tab.nl] = blocks;
                hipLaunchKernelGGL(k_col_partials, dim3(blocks), dim3(kColThreads), 0, stream, tab);
                if (int rc = launch_check("k_col_partials")) return rc;
            }
        }
        // selection for every structured layer
        {
            std::vector<int> sl;
            for (int i : ids)
                if (layers[i].kind != SA_ELEMENT) sl.push_back(i);
            for (size_t s = 0; s < sl.size(); s += kTab) {
                SelTab tab;
                memset(&tab, 0, sizeof tab);
                tab.nl = (int)std::min<size_t>(kTab, sl.size() - s);
                for (int t = 0; t < tab.nl; ++t) {
                    const sa_project_desc &d = layers[sl[s + t]];
                    const LayerPlan &p = plan[sl[s + t]];
                    SelLayer &L = tab.L[t];
                    L.partials = p.off_partials != SIZE_MAX ? ws_at<double>(ws, p.off_partials) : nullptr;
                    L.scores = d.scores ? d.scores : ws_at<double>(ws, p.off_scores);
                    L.rowpart = p.off_rowpart != SIZE_MAX ? ws_at<double>(ws, p.off_rowpart) : nullptr;
                    L.nchunk = p.rchunks;
                    L.mask = d.mask;
                    L.kept_idx = d.kept_idx;
                    L.colkeep = p.off_colkeep != SIZE_MAX ? ws_at<uint8_t>(ws, p.off_colkeep) : nullptr;
                    L.allowed = p.off_allowed != SIZE_MAX ? ws_at<uint8_t>(ws, p.off_allowed) : nullptr;
                    L.kind = d.kind;
                    L.G = (int)p.G;
                    L.k = (int)d.k;
                    L.K = p.K;
                    L.CD = p.CD;
                    L.nbands = p.nbands;
                    L.groups = d.groups;
                }
                hipLaunchKernelGGL(k_select, dim3(tab.nl), dim3(kSelThreads), 0, stream, tab);
                if (int rc = launch_check("k_select")) return rc;
            }
        }
        // element-wise layers
        {
            std::vector<int> el;
            for (int i : ids)
                if (layers[i].kind == SA_ELEMENT) el.push_back(i);
            for (size_t s = 0, step = 0; s < el.size(); s += step) {
                ElemTab tab;
                memset(&tab, 0, sizeof tab);
                step = 1;
                while (step < (size_t)kElemTab && s + step < el.size() && apart(layers, &el[s], (int)step)) ++step;
                tab.nl = (int)step;
                int blocks = 0, hblocks = 0;
                bool any = false;
                for (int t = 0; t < tab.nl; ++t) {
                    const sa_project_desc &d = layers[el[s + t]];
                    const LayerPlan &p = plan[el[s + t]];
                    ElemLayer &a = tab.L[t];
                    a.W = d.W;
                    a.U = d.U;
                    a.Z = d.Z;
                    a.G = d.G;
                    a.mask = d.mask;
                    a.kept_idx = d.kept_idx;
                    a.scores = d.scores;
                    a.inmask = held[el[s + t]] ? ws_at<uint8_t>(ws, p.off_allowed) : d.in_ch_mask;
                    char *eb = ws_at<char>(ws, p.off_elem);
                    a.hist = reinterpret_cast<uint32_t *>(eb);
                    a.state = reinterpret_cast<ElemState *>(eb + sizeof(uint32_t) * 3 * 2048);
                    a.counts = reinterpret_cast<uint2 *>(eb + sizeof(uint32_t) * 3 * 2048 + 256);
                    a.divK = make_fastdiv((uint32_t)p.K);
                    a.divAg = make_fastdiv((uint32_t)p.Ag);
                    a.divCD = make_fastdiv((uint32_t)p.CD);
                    a.n = (int32_t)(d.A * d.B * d.C * d.D);
                    a.K = p.K;
                    a.B = (int)d.B;
                    a.k = (int32_t)d.k;
                    a.sub = p.sub;
                    a.hsub = p.hsub;
                    a.rho = d.rho;
                    any = any || d.k > 0;
                    tab.begin[t] = blocks;
                    blocks += p.nblk;
                    tab.hbegin[t] = hblocks;
                    hblocks += p.hblk;
                }
                tab.begin[tab.nl] = blocks;
                tab.hbegin[tab.nl] = hblocks;
                if (any) {
                    hipLaunchKernelGGL(k_elem_init, dim3(tab.nl), dim3(kHistThreads), 0, stream, tab);
                    if (int rc = launch_check("k_elem_init")) return rc;
                    for (int pass = 0; pass < 3; ++pass) {
                        hipLaunchKernelGGL(k_elem_hist, dim3(hblocks), dim3(kHistThreads), 0, stream, tab, pass);
                        if (int rc = launch_check("k_elem_hist")) return rc;
                    }
                }
                hipLaunchKernelGGL(k_elem_count, dim3(blocks), dim3(kElemThreads), 0, stream, tab);
                if (int rc = launch_check("k_elem_count")) return rc;
                hipLaunchKernelGGL(k_elem_apply, dim3(blocks), dim3(kElemThreads), 0, stream, tab);
                if (int rc = launch_check("k_elem_apply")) return rc;
            }
        }
    }
    // apply for every structured layer, all levels at once: a level only needs
    // the masks of the levels before it, never their Z / U / G
    {
        std::vector<int> sl;
        for (int i = 0; i < n_layers; ++i)
            if (layers[i].kind != SA_ELEMENT) sl.push_back(i);
        for (size_t s = 0; s < sl.size(); s += kTab) {
            ApplyTab tab;
            memset(&tab, 0, sizeof tab);
            int blocks = 0;
            tab.nl = (int)std::min<size_t>(kTab, sl.size() - s);
            for (int t = 0; t < tab.nl; ++t) {
                RowLayer R;
                fill_row(sl[s + t], R);
                const sa_project_desc &d = layers[sl[s + t]];
                ApplyLayer &L = tab.L[t];
                L.W = R.W;
                L.U = R.U;
                L.Z = d.Z;
                L.G = d.G;
                L.rowkeep = d.kind == SA_FILTER ? d.mask : nullptr;
                L.colkeep = d.kind == SA_FILTER ? nullptr : ws_at<uint8_t>(ws, plan[sl[s + t]].off_colkeep);
                L.inmask = R.inmask;
                L.B = R.B;
                L.divCD = R.divCD;
                L.divK = make_fastdiv((uint32_t)R.K);
                L.divAg = make_fastdiv((uint32_t)R.Ag);
                L.n = (int32_t)(d.A * d.B * d.C * d.D);
                L.K = R.K;
                L.rho = R.rho;
                tab.begin[t] = blocks;
                blocks += (int)((L.n + kApplyChunk - 1) / kApplyChunk);
            }
            tab.begin[tab.nl] = blocks;
            hipLaunchKernelGGL(k_apply, dim3(blocks), dim3(kApplyThreads), 0, stream, tab);
            if (int rc = launch_check("k_apply")) return rc;
        }
    }
    return SA_OK;
}

}  // namespace
}  // namespace sa

extern "C" int structadmm_dual_update(const sa_dual_desc *layers, int n_layers, hipStream_t stream) {
    clear_error();
    if (!layers || n_layers <= 0) return fail(SA_E_ARG, "dual_update: layers must be a non-empty array");
    for (int i = 0; i < n_layers; ++i)
        if (int rc = validate_dual(layers[i], i)) return rc;
    for (int s = 0; s < n_layers; s += kTab) {
        DualTab tab;
        memset(&tab, 0, sizeof tab);
        tab.nl = std::min(kTab, n_layers - s);
        int blocks = 0;
        for (int t = 0; t < tab.nl; ++t) {
            const sa_dual_desc &d = layers[s + t];
            DualLayer &L = tab.L[t];
            L.W = d.W;
            L.Z = d.Z;
            L.U = d.U;
            L.G = d.G;
            L.n = (int32_t)d.n;
            L.update = d.update_dual ? 1 : 0;
            L.rho = d.rho;
            tab.begin[t] = blocks;
            blocks += (int)std::max<int64_t>(1, (d.n + kDualChunk - 1) / kDualChunk);
        }
        tab.begin[tab.nl] = blocks;
        hipLaunchKernelGGL(k_dual, dim3(blocks), dim3(kDualThreads), 0, stream, tab);
        if (int rc = launch_check("k_dual")) return rc;
    }
    return SA_OK;
}

extern "C" int structadmm_sgd_step(const sa_sgd_desc *layers, int n_layers, hipStream_t stream) {
    clear_error();
    if (!layers || n_layers <= 0) return fail(SA_E_ARG, "sgd_step: layers must be a non-empty array");
    for (int i = 0; i < n_layers; ++i)
        if (int rc = validate_sgd(layers[i], i)) return rc;
    for (int s = 0; s < n_layers; s += kTab) {
        SgdTab tab;
        memset(&tab, 0, sizeof tab);
        tab.nl = std::min(kTab, n_layers - s);
        int blocks = 0;
        for (int t = 0; t < tab.nl; ++t) {
            const sa_sgd_desc &d = layers[s + t];
            SgdLayer &L = tab.L[t];
            const int64_t n = d.A * d.B * d.C * d.D;
            L.W = d.W;
            L.Gf = d.Gf;
            L.Z = d.Z;
            L.U = d.U;
            L.mask = d.mask;
            L.n = (int32_t)n;
            L.kind = d.kind;
            L.divK = make_fastdiv((uint32_t)(d.B * d.C * d.D));
            L.divCD = make_fastdiv((uint32_t)(d.C * d.D));
            L.rho = d.rho;
            L.lr = d.lr;
            tab.begin[t] = blocks;
            blocks += (int)std::max<int64_t>(1, (n + kSgdChunk - 1) / kSgdChunk);
        }
        tab.begin[tab.nl] = blocks;
        hipLaunchKernelGGL(k_sgd, dim3(blocks), dim3(kSgdThreads), 0, stream, tab);
        if (int rc = launch_check("k_sgd")) return rc;
    }
    return SA_OK;
}
