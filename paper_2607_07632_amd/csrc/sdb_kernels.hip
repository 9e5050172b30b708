// Device kernels of libsdb for CDNA4 (gfx950, wave64), except the fused pass
// itself (sdb_fused.h, instantiated in sdb_fused_*.hip):
//
//  * dimension build: statistics pass, direct-mapped packed map scatter, and
//    open-addressing insert with 64-bit compare-and-swap (Section 3.3);
//  * plan sampling: each stage evaluated on its own over a strided fact sample;
//  * the fused pass's launch, the per-XCD copies' merge, the partitioned
//    terminal's passes and the sliced hash probe's partition passes;
//  * the kernel-at-a-time baselines, the streaming-read reference and
//    group-table compaction.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <climits>
#include <mutex>

#include "sdb_fused.h"

namespace sdb {
// ---------------------------------------------------------------------------
// fills
// ---------------------------------------------------------------------------

__global__ void fill_u32_kernel(uint32_t* p, uint64_t n, uint32_t v) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

__global__ void fill_u64_kernel(unsigned long long* p, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0ull;
}

__global__ void zero_pair_kernel(unsigned long long* a, unsigned long long* b, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        a[i] = 0ull;
        b[i] = 0ull;
    }
}

static int fill_grid(uint64_t n) {
    uint64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t n_words, uint32_t value, hipStream_t s) {
    if (n_words == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(fill_grid(n_words)), dim3(256), 0, s, p, n_words, value);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long* p, uint64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u64_kernel, dim3(fill_grid(n)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_zero_pair(unsigned long long* a, unsigned long long* b, uint64_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_pair_kernel, dim3(fill_grid(n)), dim3(256), 0, s, a, b, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// dimension build
// ---------------------------------------------------------------------------

__device__ __forceinline__ bool dim_row_passes(const BuildParams& bp, int64_t i) {
    bool pass = true;
    for (int q = 0; q < bp.n_preds; ++q) pass = pass && range_pass(bp.pred[q], bp.cols[bp.pred_col[q]][i]);
    return pass;
}

// The build kernels read their table's parameters in place from the batch in
// the kernel-argument segment (table = blockIdx.y).
#define SDB_BATCH_TABLE                                                                     \
    (void)kernel_args;                                                                      \
    const BuildBatch& bb = *(const BuildBatch*)__builtin_amdgcn_kernarg_segment_ptr();      \
    const BuildParams& bp = bb.bp[blockIdx.y];                                              \
    (void)bb

// Key range over all rows; pass count and payload ranges over passing rows.
// Block b of a table's stats_blocks reduces its rows in registers and LDS and
// writes its partial statistics to stats_part[b]; stats_reduce_kernel then
// combines the partials (no atomics, however many blocks).
__global__ void __launch_bounds__(256) dim_stats_kernel(BuildBatch kernel_args) {
    SDB_BATCH_TABLE;
    if ((int)blockIdx.x >= bp.stats_blocks) return;
    constexpr int kWaves = 256 / 64;
    __shared__ int32_t s_kmin[kWaves], s_kmax[kWaves], s_pkmin[kWaves], s_pkmax[kWaves];
    __shared__ unsigned long long s_np[kWaves];
    __shared__ int32_t s_pmin[SDB_MAX_PAYLOADS][kWaves], s_pmax[SDB_MAX_PAYLOADS][kWaves];
    int32_t kmin = INT_MAX, kmax = INT_MIN, pkmin = INT_MAX, pkmax = INT_MIN;
    unsigned long long npass = 0;
    int32_t pmin[SDB_MAX_PAYLOADS], pmax[SDB_MAX_PAYLOADS];
    for (int p = 0; p < SDB_MAX_PAYLOADS; ++p) {
        pmin[p] = INT_MAX;
        pmax[p] = INT_MIN;
    }
    // kBuildRows rows per thread per step, each column's loads issued together
    constexpr int U = kBuildRows;
    const int64_t stride = (int64_t)bp.stats_blocks * blockDim.x * U;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x * U + threadIdx.x; i0 < bp.n; i0 += stride) {
        bool ok[U], pass[U];
        int32_t x[U], key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + (int64_t)u * blockDim.x;
            ok[u] = i < bp.n;
            key[u] = ok[u] ? bp.key[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (ok[u]) {
                kmin = min(kmin, key[u]);
                kmax = max(kmax, key[u]);
            }
            pass[u] = ok[u];
        }
        for (int q = 0; q < bp.n_preds; ++q) {
            const int32_t* col = bp.cols[bp.pred_col[q]];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = ok[u] ? col[i0 + (int64_t)u * blockDim.x] : 0;
#pragma unroll
            for (int u = 0; u < U; ++u) pass[u] = pass[u] && range_pass(bp.pred[q], x[u]);
        }
        for (int p = 0; p < bp.n_payloads; ++p) {
            const int32_t* col = bp.cols[bp.payload_col[p]];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = pass[u] ? col[i0 + (int64_t)u * blockDim.x] : 0;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (pass[u]) {
                    pmin[p] = min(pmin[p], x[u]);
                    pmax[p] = max(pmax[p], x[u]);
                }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            npass += pass[u] ? 1ull : 0ull;
            if (pass[u]) {
                pkmin = min(pkmin, key[u]);
                pkmax = max(pkmax, key[u]);
            }
        }
    }
    kmin = wave_min_i32(kmin);
    kmax = wave_max_i32(kmax);
    pkmin = wave_min_i32(pkmin);
    pkmax = wave_max_i32(pkmax);
    npass = wave_sum_u64(npass);
    for (int p = 0; p < SDB_MAX_PAYLOADS; ++p) {
        pmin[p] = wave_min_i32(pmin[p]);
        pmax[p] = wave_max_i32(pmax[p]);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_kmin[wave] = kmin;
        s_kmax[wave] = kmax;
        s_pkmin[wave] = pkmin;
        s_pkmax[wave] = pkmax;
        s_np[wave] = npass;
        for (int p = 0; p < SDB_MAX_PAYLOADS; ++p) {
            s_pmin[p][wave] = pmin[p];
            s_pmax[p][wave] = pmax[p];
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kWaves; ++w) {
            kmin = min(kmin, s_kmin[w]);
            kmax = max(kmax, s_kmax[w]);
            pkmin = min(pkmin, s_pkmin[w]);
            pkmax = max(pkmax, s_pkmax[w]);
            npass += s_np[w];
            for (int p = 0; p < SDB_MAX_PAYLOADS; ++p) {
                pmin[p] = min(pmin[p], s_pmin[p][w]);
                pmax[p] = max(pmax[p], s_pmax[p][w]);
            }
        }
        DimStats part;
        part.kmin = kmin;
        part.kmax = kmax;
        part.npass = npass;
        for (int p = 0; p < SDB_MAX_PAYLOADS; ++p) {
            part.pmin[p] = pmin[p];
            part.pmax[p] = pmax[p];
        }
        part.dup = 0u;
        part.pad_ = 0u;
        part.occupied = 0ull;
        part.pkmin = pkmin;
        part.pkmax = pkmax;
        bp.stats_part[blockIdx.x] = part;
    }
}

// One block per table: the table's statistics from its blocks' partials
// (and the duplicate and occupancy counters the build passes add to, zeroed).
__global__ void __launch_bounds__(256) stats_reduce_kernel(BuildBatch kernel_args) {
    SDB_BATCH_TABLE;
    __shared__ DimStats red[256 / 64];
    DimStats acc;
    acc.kmin = INT_MAX;
    acc.kmax = INT_MIN;
    acc.npass = 0ull;
    for (int p = 0; p < SDB_MAX_PAYLOADS; ++p) {
        acc.pmin[p] = INT_MAX;
        acc.pmax[p] = INT_MIN;
    }
    acc.dup = 0u;
    acc.pad_ = 0u;
    acc.occupied = 0ull;
    acc.pkmin = INT_MAX;
    acc.pkmax = INT_MIN;
    // up to kStatsMaxBlocks / 256 partials per thread, loaded together
    constexpr int kPer = kStatsMaxBlocks / 256;
    static_assert(kPer * 256 == kStatsMaxBlocks, "whole partials per thread");
    DimStats part[kPer];
    bool have[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int b = (int)threadIdx.x + u * 256;
        have[u] = b < bp.stats_blocks;
        if (have[u]) part[u] = bp.stats_part[b];
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (!have[u]) continue;
        const DimStats& s = part[u];
        acc.kmin = min(acc.kmin, s.kmin);
        acc.kmax = max(acc.kmax, s.kmax);
        acc.npass += s.npass;
        acc.pkmin = min(acc.pkmin, s.pkmin);
        acc.pkmax = max(acc.pkmax, s.pkmax);
        for (int p = 0; p < SDB_MAX_PAYLOADS; ++p) {
            acc.pmin[p] = min(acc.pmin[p], s.pmin[p]);
            acc.pmax[p] = max(acc.pmax[p], s.pmax[p]);
        }
    }
    // wave reductions, then the 4 waves' results in LDS
    acc.kmin = wave_min_i32(acc.kmin);
    acc.kmax = wave_max_i32(acc.kmax);
    acc.npass = wave_sum_u64(acc.npass);
    acc.pkmin = wave_min_i32(acc.pkmin);
    acc.pkmax = wave_max_i32(acc.pkmax);
    for (int p = 0; p < SDB_MAX_PAYLOADS; ++p) {
        acc.pmin[p] = wave_min_i32(acc.pmin[p]);
        acc.pmax[p] = wave_max_i32(acc.pmax[p]);
    }
    if ((threadIdx.x & 63u) == 0u) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        DimStats a = red[0];
        for (uint32_t w = 1; w < blockDim.x / 64u; ++w) {
            const DimStats& s = red[w];
            a.kmin = min(a.kmin, s.kmin);
            a.kmax = max(a.kmax, s.kmax);
            a.npass += s.npass;
            a.pkmin = min(a.pkmin, s.pkmin);
            a.pkmax = max(a.pkmax, s.pkmax);
            for (int p = 0; p < SDB_MAX_PAYLOADS; ++p) {
                a.pmin[p] = min(a.pmin[p], s.pmin[p]);
                a.pmax[p] = max(a.pmax[p], s.pmax[p]);
            }
        }
        *bp.stats = a;
        if (bb.host_stats) bb.host_stats[blockIdx.y] = a;
    }
}

// One block: every table's statistics block, word by word, to pinned host memory.
__global__ void __launch_bounds__(256) export_stats_kernel(BuildBatch kernel_args) {
    (void)kernel_args;
    const BuildBatch& bb = *(const BuildBatch*)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int kWords = sizeof(DimStats) / 4;
    for (int i = threadIdx.x; i < bb.n * kWords; i += blockDim.x) {
        const uint32_t* src = reinterpret_cast<const uint32_t*>(bb.bp[i / kWords].stats);
        reinterpret_cast<uint32_t*>(bb.host_stats + i / kWords)[i % kWords] = src[i % kWords];
    }
}

__global__ void __launch_bounds__(256) copy_out_kernel(const uint32_t* src0, uint32_t words0, const uint32_t* src1,
                                                       uint32_t words1, uint32_t* dst) {
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < words0 + words1; i += stride)
        dst[i] = i < words0 ? src0[i] : src1[i - words0];
}

__device__ __forceinline__ uint32_t dim_row_code(const BuildParams& bp, int64_t i) {
    uint32_t c = 0;
    for (int p = 0; p < bp.n_payloads; ++p)
        c += (uint32_t)(bp.cols[bp.payload_col[p]][i] - bp.pmin[p]) * bp.pdiv[p];
    return c;
}

// Direct-mapped map over the keys [kmin, kmin + nslots): the fill leaves
// every slot at `missing` (all ones: no row holds the key); a passing row then
// stores its code and a filtered row the sentinel (`missing` - 1). Plain
// stores, no atomics: each key owns its slot.
__global__ void __launch_bounds__(256) fill_table_kernel(BuildBatch kernel_args) {
    SDB_BATCH_TABLE;
    uint32_t* w = static_cast<uint32_t*>(bp.map);
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < bp.fill_words; i += stride)
        w[i] = bp.fill_value;
}

__global__ void __launch_bounds__(256) dense_scatter_kernel(BuildBatch kernel_args) {
    SDB_BATCH_TABLE;
    if (!bp.dense) return;
    // kBuildRows rows per thread per step, each column's loads issued together
    // (a row at a time, the key, predicate and payload loads form one chain)
    constexpr int U = kBuildRows;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x * U;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x * U + threadIdx.x; i0 < bp.n; i0 += stride) {
        bool ok[U], pass[U];
        int32_t x[U];
        uint32_t idx[U], code[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + (int64_t)u * blockDim.x;
            ok[u] = i < bp.n;
            x[u] = ok[u] ? bp.key[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            idx[u] = (uint32_t)((int64_t)x[u] - (int64_t)bp.kmin);
            pass[u] = ok[u];
            code[u] = 0u;
        }
        for (int q = 0; q < bp.n_preds; ++q) {
            const int32_t* col = bp.cols[bp.pred_col[q]];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = ok[u] ? col[i0 + (int64_t)u * blockDim.x] : 0;
#pragma unroll
            for (int u = 0; u < U; ++u) pass[u] = pass[u] && range_pass(bp.pred[q], x[u]);
        }
        for (int p = 0; p < bp.n_payloads; ++p) {
            const int32_t* col = bp.cols[bp.payload_col[p]];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = pass[u] ? col[i0 + (int64_t)u * blockDim.x] : 0;
#pragma unroll
            for (int u = 0; u < U; ++u) code[u] += (uint32_t)((int64_t)x[u] - (int64_t)bp.pmin[p]) * bp.pdiv[p];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!ok[u]) continue;
            if ((uint64_t)idx[u] >= bp.nslots) {          // cannot happen: kmin/kmax cover all keys
                atomicOr(&bp.stats->dup, 4u);
                continue;
            }
            const uint32_t c = pass[u] ? code[u] : bp.sentinel;
            if (bp.width == 1) static_cast<uint8_t*>(bp.map)[idx[u]] = (uint8_t)c;
            else if (bp.width == 2) static_cast<uint16_t*>(bp.map)[idx[u]] = (uint16_t)c;
            else static_cast<uint32_t*>(bp.map)[idx[u]] = c;
        }
    }
}

// One thread per 32 slots: the pass bitmap word (code below the sentinel)
// and the number of occupied slots. Distinct keys occupy n slots; a duplicate
// key leaves fewer, which the host detects from the total.
__global__ void __launch_bounds__(256) dense_bits_kernel(BuildBatch kernel_args) {
    SDB_BATCH_TABLE;
    if (!bp.dense) return;
    const uint64_t n_words = (bp.nslots + 31) / 32;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    unsigned long long occupied = 0;
    for (uint64_t w = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; w < n_words; w += stride) {
        // the word's 32 map entries as 16-byte loads (the map is padded to 256
        // bytes and filled, so the last word's loads stay inside it)
        uint32_t bits = 0u;
        const uint32_t valid = (uint32_t)min<uint64_t>(32, bp.nslots - w * 32);
        if (bp.width == 1) {
            const v4u* src = reinterpret_cast<const v4u*>(static_cast<const uint8_t*>(bp.map) + w * 32);
            const v4u a = src[0], b = src[1];
            const uint32_t d[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (uint32_t e = 0; e < 32u; ++e) {
                const uint32_t c = (d[e >> 2] >> ((e & 3u) * 8u)) & 0xFFu;
                if (e < valid) {
                    bits |= (c < bp.sentinel ? 1u : 0u) << e;
                    occupied += c != bp.missing;
                }
            }
        } else if (bp.width == 2) {
            const v4u* src = reinterpret_cast<const v4u*>(static_cast<const uint16_t*>(bp.map) + w * 32);
            uint32_t d[16];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const v4u a = src[k];
                d[4 * k] = a.x;
                d[4 * k + 1] = a.y;
                d[4 * k + 2] = a.z;
                d[4 * k + 3] = a.w;
            }
#pragma unroll
            for (uint32_t e = 0; e < 32u; ++e) {
                const uint32_t c = (d[e >> 1] >> ((e & 1u) * 16u)) & 0xFFFFu;
                if (e < valid) {
                    bits |= (c < bp.sentinel ? 1u : 0u) << e;
                    occupied += c != bp.missing;
                }
            }
        } else {
            const v4u* src = reinterpret_cast<const v4u*>(static_cast<const uint32_t*>(bp.map) + w * 32);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const v4u a = src[k];
                const uint32_t d[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
                for (uint32_t e4 = 0; e4 < 4u; ++e4) {
                    const uint32_t e = (uint32_t)k * 4u + e4;
                    if (e < valid) {
                        bits |= (d[e4] < bp.sentinel ? 1u : 0u) << e;
                        occupied += d[e4] != bp.missing;
                    }
                }
            }
        }
        bp.pass_bits[w] = bits;
    }
    occupied = wave_sum_u64(occupied);
    __shared__ unsigned long long s_occ[4];
    if ((threadIdx.x & 63) == 0) s_occ[threadIdx.x >> 6] = occupied;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long t = s_occ[0] + s_occ[1] + s_occ[2] + s_occ[3];
        if (t) atomicAdd(&bp.stats->occupied, t);
    }
}

// The slot value of dimension row i: {key, code + 1 | 0xFFFFFFFF}.
__device__ __forceinline__ unsigned long long hash_slot_value(const BuildParams& bp, int64_t i) {
    const uint32_t enc = dim_row_passes(bp, i) ? dim_row_code(bp, i) + 1u : 0xFFFFFFFFu;
    return ((unsigned long long)enc << 32) | (uint32_t)bp.key[i];
}

// A passing row's key goes into the table's pass filter.
__device__ __forceinline__ void hash_filter_key(const BuildParams& bp, unsigned long long slot) {
    uint32_t fw, fm;
    if (bp.filt && !bp.filt_via_bytes && (uint32_t)(slot >> 32) != 0xFFFFFFFFu &&
        filter_slot(bp.filt_kind, bp.filt_bits, bp.kmin, (int32_t)(uint32_t)slot, fw, fm))
        atomicOr(&bp.filt[fw], fm);
}

// Open addressing, linear probing, 8-byte slots.
__device__ __forceinline__ void hash_place(const BuildParams& bp, unsigned long long slot) {
    unsigned long long* tab = static_cast<unsigned long long*>(bp.map);
    const uint32_t k = (uint32_t)slot;
    uint32_t h = (k * 0x9E3779B1u) >> bp.hshift & bp.hmask;
    for (uint64_t it = 0; it < bp.nslots; ++it) {
        const unsigned long long old = atomicCAS(&tab[h], 0ull, slot);
        if (old == 0ull) return;
        if ((uint32_t)old == k) {
            atomicOr(&bp.stats->dup, 1u);
            return;
        }
        h = (h + 1u) & bp.hmask;
    }
    atomicOr(&bp.stats->dup, 2u);
}

__global__ void __launch_bounds__(256) hash_insert_kernel(BuildBatch kernel_args) {
    SDB_BATCH_TABLE;
    if (bp.dense || bp.sliced) return;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < bp.n; i += stride) {
        const unsigned long long slot = hash_slot_value(bp, i);
        hash_filter_key(bp, slot);
        hash_place(bp, slot);
    }
}

// A hash table's pass bitmap without atomics (filt_via_bytes): the slot
// region, not yet filled, first holds one byte per key of the range, cleared,
// then set by every passing row with a plain store; the bytes are then
// packed 32 to a filter word. Each key has its own byte, so no two rows
// write the same address unless they hold the same key (a duplicate, which
// the inserts report).
__global__ void __launch_bounds__(256) filter_clear_kernel(BuildBatch kernel_args) {
    SDB_BATCH_TABLE;
    if (!bp.filt_via_bytes) return;
    uint32_t* w = static_cast<uint32_t*>(bp.map);
    const uint64_t n_words = (bp.filt_bits + 31u) / 32u * 8u;   // the bytes the packing reads
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words; i += stride) w[i] = 0u;
}

__global__ void __launch_bounds__(256) filter_mark_kernel(BuildBatch kernel_args) {
    SDB_BATCH_TABLE;
    if (!bp.filt_via_bytes) return;
    uint8_t* b = static_cast<uint8_t*>(bp.map);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < bp.n; i += stride) {
        const uint32_t idx = (uint32_t)bp.key[i] - (uint32_t)bp.kmin;
        if ((uint64_t)idx < bp.filt_bits && dim_row_passes(bp, i)) b[idx] = 1u;
    }
}

__global__ void __launch_bounds__(256) filter_pack_kernel(BuildBatch kernel_args) {
    SDB_BATCH_TABLE;
    if (!bp.filt_via_bytes) return;
    const v4u* b = static_cast<const v4u*>(bp.map);
    const uint64_t n_words = (bp.filt_bits + 31u) / 32u;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t w = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; w < n_words; w += stride) {
        const v4u lo = b[2 * w], hi = b[2 * w + 1];   // the 32 key bytes of word w
        const uint32_t q[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        uint32_t out = 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if ((q[j] >> (8 * t)) & 0xFFu) out |= 1u << (4 * j + t);
        if (32u * w + 32u > bp.filt_bits) out &= (1u << (uint32_t)(bp.filt_bits - 32u * w)) - 1u;   // past the range
        bp.filt[w] = out;
    }
}

static int build_grid(int64_t n) {
    int64_t g = (n + 255) / 256;
    if (g > 2048) g = 2048;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_build_stats(const BuildBatch& bb, hipStream_t s) {
    if (bb.n <= 0) return hipSuccess;
    int g = 1;
    for (int d = 0; d < bb.n; ++d) {
        if (bb.bp[d].stats_blocks < 1 || bb.bp[d].stats_blocks > kStatsMaxBlocks) return hipErrorInvalidValue;
        g = std::max(g, bb.bp[d].stats_blocks);
    }
    hipLaunchKernelGGL(dim_stats_kernel, dim3(g, bb.n), dim3(256), 0, s, bb);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(stats_reduce_kernel, dim3(1, bb.n), dim3(256), 0, s, bb);
    return hipGetLastError();
}

hipError_t launch_export_stats(const BuildBatch& bb, hipStream_t s) {
    if (bb.n <= 0) return hipSuccess;
    if (!bb.host_stats || bb.n > SDB_MAX_JOINS) return hipErrorInvalidValue;
    hipLaunchKernelGGL(export_stats_kernel, dim3(1), dim3(256), 0, s, bb);
    return hipGetLastError();
}

hipError_t launch_copy_out(const uint32_t* src0, uint32_t words0, const uint32_t* src1, uint32_t words1,
                           uint32_t* dst, hipStream_t s) {
    const uint64_t total = (uint64_t)words0 + words1;
    if (total == 0) return hipSuccess;
    if (!dst || (words0 && !src0) || (words1 && !src1) || total > (1ull << 30)) return hipErrorInvalidValue;
    uint64_t g = (total + 255) / 256;
    if (g > 64) g = 64;
    hipLaunchKernelGGL(copy_out_kernel, dim3((uint32_t)g), dim3(256), 0, s, src0, words0, src1, words1, dst);
    return hipGetLastError();
}

hipError_t launch_build_tables(const BuildBatch& bb, hipStream_t s) {
    if (bb.n <= 0) return hipSuccess;
    uint64_t words = 0, n_words32 = 0, filt_words = 0;
    int64_t n_dense = 0, n_hash = 0, n_filt = 0;
    for (int d = 0; d < bb.n; ++d) {
        const BuildParams& bp = bb.bp[d];
        words = std::max<uint64_t>(words, bp.fill_words);
        if (bp.dense) {
            n_dense = std::max<int64_t>(n_dense, bp.n);
            n_words32 = std::max<uint64_t>(n_words32, (bp.nslots + 31) / 32);
        } else if (!bp.sliced) {
            n_hash = std::max<int64_t>(n_hash, bp.n);
        }
        if (bp.filt_via_bytes) {
            n_filt = std::max<int64_t>(n_filt, bp.n);
            filt_words = std::max<uint64_t>(filt_words, (bp.filt_bits + 31) / 32);
        }
    }
    if (filt_words > 0) {   // before the fill: the bytes live in the slot region
        hipLaunchKernelGGL(filter_clear_kernel, dim3(fill_grid(filt_words * 8), bb.n), dim3(256), 0, s, bb);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (n_filt > 0) {
            hipLaunchKernelGGL(filter_mark_kernel, dim3(build_grid(n_filt), bb.n), dim3(256), 0, s, bb);
            e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(filter_pack_kernel, dim3(fill_grid(filt_words), bb.n), dim3(256), 0, s, bb);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (words > 0) {
        hipLaunchKernelGGL(fill_table_kernel, dim3(fill_grid(words), bb.n), dim3(256), 0, s, bb);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n_dense > 0) {
        hipLaunchKernelGGL(dense_scatter_kernel, dim3(build_grid((n_dense + kBuildRows - 1) / kBuildRows), bb.n),
                           dim3(256), 0, s, bb);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n_words32 > 0) {
        hipLaunchKernelGGL(dense_bits_kernel, dim3(build_grid((int64_t)n_words32), bb.n), dim3(256), 0, s, bb);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (n_hash > 0) {
        hipLaunchKernelGGL(hash_insert_kernel, dim3(build_grid(n_hash), bb.n), dim3(256), 0, s, bb);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---------------------------------------------------------------------------
// coarse pass bitmap of a dense table (LDS_COARSE placement)
// ---------------------------------------------------------------------------

// Thread w writes coarse word w: bit b is set iff one of the 2^shift slots
// starting at slot (32 w + b) << shift passes. 2^shift divides 32, so every
// group of slots lies inside one word of the pass bitmap.
__global__ void __launch_bounds__(256) coarse_bits_kernel(CoarseParams cp) {
    const uint32_t w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= cp.n_words) return;
    const uint32_t per = 1u << cp.shift;
    const uint32_t mask = per >= 32u ? 0xFFFFFFFFu : ((1u << per) - 1u);
    const uint32_t n_fine = (cp.nslots + 31u) / 32u;
    uint32_t out = 0u;
    for (uint32_t b = 0; b < 32u; ++b) {
        const uint64_t first = ((uint64_t)w * 32u + b) << cp.shift;
        if (first >= cp.nslots) break;
        const uint32_t fw = (uint32_t)(first >> 5);
        const uint32_t word = fw < n_fine ? cp.bits[fw] : 0u;
        if ((word >> (uint32_t)(first & 31u)) & mask) out |= 1u << b;
    }
    cp.out[w] = out;
}

hipError_t launch_coarse_build(const CoarseParams& cp, hipStream_t s) {
    if (cp.n_words == 0) return hipSuccess;
    hipLaunchKernelGGL(coarse_bits_kernel, dim3((cp.n_words + 255u) / 256u), dim3(256), 0, s, cp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// rank tables of a dense table (LDS_RANK placement)
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint32_t rank_word(const RankParams& rp, uint32_t w) {
    return w < (rp.nslots + 31u) / 32u ? rp.bits[w] : 0u;
}

constexpr uint32_t kRankWords = 256;   // bitmap words per block, one per thread

// Block b < rank_blocks: words 256 b .. of the bitmap. It counts the passing
// slots of all words before (at most 8,192 words, an L2 read of 32 KB), scans
// its own, writes the 64-slot groups' counts and stores the passing slots'
// codes at their ranks. The other blocks zero the outputs: one launch in place
// of three (about 4.5 us each when launches follow one another).
__global__ void __launch_bounds__(256) rank_build_kernel(RankParams rp, uint32_t rank_blocks) {
    if (blockIdx.x >= rank_blocks) {
        const uint64_t stride = (uint64_t)(gridDim.x - rank_blocks) * 256u;
        for (uint64_t i = (uint64_t)(blockIdx.x - rank_blocks) * 256u + threadIdx.x; i < rp.zero_n; i += stride) {
            rp.zero_a[i] = 0ull;
            rp.zero_b[i] = 0ull;
        }
        return;
    }
    __shared__ uint32_t wbefore[4], wown[4], wbits[kRankWords], wrank[kRankWords];
    const uint32_t w0 = blockIdx.x * kRankWords, w = w0 + threadIdx.x;
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t before = 0;
    const v4u* quads = reinterpret_cast<const v4u*>(rp.bits);   // (whole quads: w0 is a multiple of 256)
#pragma unroll 8
    for (uint32_t i = threadIdx.x; i < w0 / 4u; i += kRankWords) {
        const v4u x = quads[i];
        before += (uint32_t)(__popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w));
    }
    for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off, 64);
    const uint32_t bits = rank_word(rp, w);
    const uint32_t own = (uint32_t)__popc(bits);
    uint32_t x = own;
    for (uint32_t off = 1; off < 64u; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63u) {
        wbefore[wave] = before;
        wown[wave] = x;
    }
    __syncthreads();
    uint32_t r = x - own + wbefore[0] + wbefore[1] + wbefore[2] + wbefore[3];
    for (uint32_t v = 0; v < wave; ++v) r += wown[v];
    if ((w & 1u) == 0u && w / 2u < (rp.nslots + 63u) / 64u) rp.prefix[w / 2u] = r;
    wbits[threadIdx.x] = bits;
    wrank[threadIdx.x] = r;
    __syncthreads();
    // a thread per slot, all its 32 slots' codes read together
    uint32_t c[32];
#pragma unroll
    for (uint32_t u = 0; u < 32u; ++u) {
        const uint32_t slot = min(w0 * 32u + u * 256u + threadIdx.x, rp.nslots - 1u);
        if (rp.width == 1) c[u] = static_cast<const uint8_t*>(rp.map)[slot];
        else if (rp.width == 2) c[u] = static_cast<const uint16_t*>(rp.map)[slot];
        else c[u] = static_cast<const uint32_t*>(rp.map)[slot];
    }
#pragma unroll
    for (uint32_t u = 0; u < 32u; ++u) {   // (bits past the last slot are clear)
        const uint32_t i = u * 8u + (threadIdx.x >> 5), bit = threadIdx.x & 31u;
        if (!((wbits[i] >> bit) & 1u)) continue;
        const uint32_t to = wrank[i] + (uint32_t)__popc(wbits[i] & ((1u << bit) - 1u));
        if (rp.width == 1) static_cast<uint8_t*>(rp.codes)[to] = (uint8_t)c[u];
        else if (rp.width == 2) static_cast<uint16_t*>(rp.codes)[to] = (uint16_t)c[u];
        else static_cast<uint32_t*>(rp.codes)[to] = c[u];
    }
}

hipError_t launch_rank_build(const RankParams& rp, hipStream_t s) {
    if (rp.nslots == 0 || (rp.nslots + 63u) / 64u > kRankGroups) return hipErrorInvalidValue;
    const uint32_t blocks = ((rp.nslots + 31u) / 32u + kRankWords - 1u) / kRankWords;
    const uint32_t zero = rp.zero_n ? (uint32_t)std::min<uint64_t>(1024u, (rp.zero_n + 255u) / 256u) : 0u;
    hipLaunchKernelGGL(rank_build_kernel, dim3(blocks + zero), dim3(256), 0, s, rp, blocks);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// plan sampling: pass count of every stage on its own over a strided sample
// ---------------------------------------------------------------------------

// Every sampled row (row k * step) is evaluated against every stage on its
// own; the pattern of stages it passes (bit s for stage s) is counted in
// pattern_hist, and for a dense-table stage the bucket of its key in the
// table's key range (kKeyBuckets equal buckets) in key_hist[s].
__global__ void __launch_bounds__(256) sample_kernel(FusedParams kernel_args, int64_t step, int64_t n_sample,
                                                     int32_t n_ranges, uint32_t* pattern_hist, uint32_t* key_hist) {
    (void)kernel_args;
    const FusedParams& p = *(const FusedParams*)__builtin_amdgcn_kernarg_segment_ptr();
    // block-private histograms in LDS (the few pass patterns of a small plan
    // would otherwise draw every sampled row's atomic onto a handful of words)
    __shared__ uint32_t kh[kMaxStages * kKeyBuckets];
    __shared__ uint32_t ph[kSamplePatternsLds];
    const uint32_t n_patterns = (uint32_t)n_ranges << p.nstages;
    const bool lds_patterns = n_patterns <= (uint32_t)kSamplePatternsLds;
    for (int i = threadIdx.x; i < p.nstages * kKeyBuckets; i += blockDim.x) kh[i] = 0u;
    for (uint32_t i = threadIdx.x; lds_patterns && i < n_patterns; i += blockDim.x) ph[i] = 0u;
    __syncthreads();
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n_sample; k += stride) {
        const int64_t row = k * step;
        uint32_t pattern = 0u;
        for (int s = 0; s < p.nstages; ++s) {
            const StageDev& S = p.st[s];
            const int32_t x = p.cols[S.col][row];
            if (stage_pass_one(S, x)) pattern |= 1u << s;
            if (S.sample_hist && S.kind == ST_DENSE && S.nslots > 0u) {
                const uint32_t idx = (uint32_t)(x - S.kmin);
                if (idx < S.nslots)
                    atomicAdd(&kh[s * kKeyBuckets + (uint32_t)((uint64_t)idx * kKeyBuckets / S.nslots)], 1u);
            }
        }
        const uint32_t bin = (uint32_t)(k * n_ranges / n_sample) << p.nstages | pattern;
        if (lds_patterns) atomicAdd(&ph[bin], 1u);
        else atomicAdd(&pattern_hist[bin], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < p.nstages * kKeyBuckets; i += blockDim.x)
        if (kh[i]) atomicAdd(&key_hist[i], kh[i]);
    for (uint32_t i = threadIdx.x; lds_patterns && i < n_patterns; i += blockDim.x)
        if (ph[i]) atomicAdd(&pattern_hist[i], ph[i]);
}

hipError_t launch_sample(const FusedParams& p, int64_t step, int64_t n_sample, int32_t n_ranges,
                         uint32_t* pattern_hist, uint32_t* key_hist, hipStream_t s) {
    if (p.nstages < 0 || p.nstages > kMaxStages || n_ranges < 1 || ((uint64_t)n_ranges << p.nstages) > (1ull << kMaxStages))
        return hipErrorInvalidValue;
    hipError_t e;
    if (key_hist == pattern_hist + (1u << kMaxStages)) {
        e = launch_fill_u32(pattern_hist, (1u << kMaxStages) + (uint64_t)kMaxStages * kKeyBuckets, 0u, s);
    } else {
        e = launch_fill_u32(pattern_hist, (uint64_t)n_ranges << p.nstages, 0u, s);
        if (e != hipSuccess) return e;
        e = launch_fill_u32(key_hist, (uint64_t)kMaxStages * kKeyBuckets, 0u, s);
    }
    if (e != hipSuccess || n_sample == 0 || p.nstages == 0) return e;
    int64_t g = (n_sample + 255) / 256;
    if (g > 256) g = 256;
    hipLaunchKernelGGL(sample_kernel, dim3((int)g), dim3(256), 0, s, p, step, n_sample, n_ranges, pattern_hist,
                       key_hist);
    return hipGetLastError();
}

// Adds the per-XCD copies into the outputs (which it overwrites).
__global__ void __launch_bounds__(256) xcd_merge_kernel(const unsigned long long* xtab, int copies,
                                                        uint64_t n_groups, unsigned long long* sums,
                                                        unsigned long long* counts) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_groups; g += stride) {
        unsigned long long s = 0, c = 0;
        for (int x = 0; x < copies; ++x) {
            const unsigned long long* e = xtab + 2ull * (n_groups * (uint64_t)x + g);
            s += e[0];
            c += e[1];
        }
        sums[g] = s;
        counts[g] = c;
    }
}

hipError_t launch_xcd_merge(const unsigned long long* xtab, int copies, uint64_t n_groups,
                            unsigned long long* sums, unsigned long long* counts, hipStream_t s) {
    if (n_groups == 0) return hipSuccess;
    hipLaunchKernelGGL(xcd_merge_kernel, dim3(fill_grid(n_groups)), dim3(256), 0, s, xtab, copies, n_groups,
                       sums, counts);
    return hipGetLastError();
}


// Instances: 4-row or 1-row items, 1/2/4 items per lane, every terminal;
// eager column loads for 4-row items with 1 or 2 items per lane; blocks of
// kBigBlock threads for 4-row items with 1 or 2 items per lane; the stage
// loop written out kUnrollStages times for 4-row items, 2 items per lane,
// blocks of kMaxBlock or kBigBlock and no eager loads.
static const void* pick_fused(int vector, int ipt, int terminal, int eager, int block, int unroll) {
    if (unroll < 0) return vector && eager <= 0 && block <= kBigBlock ? pick_fused_probe(ipt, terminal) : nullptr;
    if (unroll) {
        if (!vector || ipt != 2 || eager > 0) return nullptr;
        if (block <= kMaxBlock) return pick_fused_unrolled(terminal);
        if (block == kBigBlock) return pick_fused_unrolled_big(terminal);
        return nullptr;
    }
    if (block == kBigBlock) return vector && eager <= 0 ? pick_fused_big(ipt, terminal) : nullptr;
    if (block > kMaxBlock) return nullptr;
    if (eager > 0) return vector ? pick_fused_eager(ipt, terminal) : nullptr;
    return vector ? pick_fused_vec(ipt, terminal) : pick_fused_rows(ipt, terminal);
}

int fused_blocks_per_cu(int vector, int ipt, int terminal, int eager, int block, int unroll, size_t lds_bytes) {
    const void* fn = pick_fused(vector, ipt, terminal, eager, block, unroll);
    if (!fn) return -1;
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, fn, block, lds_bytes) != hipSuccess)
        return -1;
    return blocks;
}

hipError_t launch_fused(const FusedParams& p, int vector, int ipt, int terminal, int eager, int unroll, int grid,
                        int block, size_t lds_bytes, hipStream_t s) {
    if (unroll > 0 && p.nstages > kUnrollStages) return hipErrorInvalidValue;
    const void* fn = pick_fused(vector, ipt, terminal, eager, block, unroll);
    if (!fn) return hipErrorInvalidValue;
    void* args[] = {const_cast<FusedParams*>(&p)};
    return hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds_bytes, s);
}


// ---------------------------------------------------------------------------
// kernel-at-a-time execution: one kernel per operator, flags and group ids in
// global memory between them (the unfused baseline)
// ---------------------------------------------------------------------------

struct UnfusedParams {
    const int32_t* col;        // the stage's fact column (stage kernels), agg operand a (aggregate kernel)
    const int32_t* col_b;      // agg operand b
    int64_t n;
    uint8_t* flags;            // live flag per row
    uint32_t* gid;             // group id per row
    unsigned long long* sums;
    unsigned long long* counts;
    int32_t agg_kind;
    int32_t pad_;
    StageDev st;
};

__global__ void __launch_bounds__(256) unfused_init_kernel(UnfusedParams up) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < up.n; i += stride) {
        up.flags[i] = 1u;
        up.gid[i] = 0u;
    }
}

// One row of one stage with its table in device memory: whether the row
// passes, and the dimension code it gathers (pass implies c < sentinel).
__device__ __forceinline__ bool device_stage_row(const StageDev& S, int32_t x, uint32_t& c) {
    c = 0u;
    if (S.kind == ST_PRED) return range_pass(S.test, x);
    if (S.kind == ST_DENSE) {
        const uint32_t idx = (uint32_t)(x - S.kmin);
        if (idx >= S.nslots) return false;
        c = load_dense_code(S, idx);
        return c < S.sentinel;
    }
    const uint32_t h = hash_slot(S, x);
    c = hash_resolve(S, x, h, static_cast<const unsigned long long*>(S.map)[h]);
    return c < S.sentinel;
}

// The part of the mixed-radix group id that a passing row's code adds.
__device__ __forceinline__ uint32_t stage_gid_part(const StageDev& S, uint32_t c) {
    if (S.gk_mode == GK_ONE) return c * S.gk_stride[0];
    if (S.gk_mode == GK_GENERAL) return code_contribution(S, c);
    return 0u;
}

__device__ __forceinline__ long long row_value(int32_t kind, int32_t a, int32_t b) {
    const long long x = a;
    if (kind == SDB_AGG_MUL) return x * (long long)b;
    if (kind == SDB_AGG_SUB) return x - (long long)b;
    if (kind == SDB_AGG_ADD) return x + (long long)b;
    return x;
}

// One stage over every row still flagged: predicate, dense map or hash probe.
__global__ void __launch_bounds__(256) unfused_stage_kernel(UnfusedParams kernel_args) {
    (void)kernel_args;
    const UnfusedParams& up = *(const UnfusedParams*)__builtin_amdgcn_kernarg_segment_ptr();
    const StageDev& S = up.st;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < up.n; i += stride) {
        if (!up.flags[i]) continue;
        uint32_t c;
        if (!device_stage_row(S, up.col[i], c)) up.flags[i] = 0u;
        else if (S.gk_mode != GK_NONE) up.gid[i] += stage_gid_part(S, c);
    }
}

// The aggregate of every flagged row, added into the outputs with atomics.
__global__ void __launch_bounds__(256) unfused_agg_kernel(UnfusedParams up) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < up.n; i += stride) {
        if (!up.flags[i]) continue;
        const long long v = row_value(up.agg_kind, up.col[i], up.col_b[i]);
        const uint32_t g = up.gid[i];
        atomicAdd(&up.sums[g], (unsigned long long)v);
        atomicAdd(&up.counts[g], 1ull);
    }
}

static int unfused_grid(int64_t n) {
    int64_t g = (n + 255) / 256;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_unfused(const FusedParams& p, uint8_t* flags, uint32_t* gid, hipStream_t s) {
    if (p.n == 0) return hipSuccess;
    UnfusedParams up;
    memset(&up, 0, sizeof up);
    up.n = p.n;
    up.flags = flags;
    up.gid = gid;
    up.sums = p.sums;
    up.counts = p.counts;
    up.agg_kind = p.agg_kind;
    const int grid = unfused_grid(p.n);
    hipLaunchKernelGGL(unfused_init_kernel, dim3(grid), dim3(256), 0, s, up);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int st = 0; st < p.nstages; ++st) {
        up.st = p.st[st];
        up.col = p.cols[up.st.col];
        hipLaunchKernelGGL(unfused_stage_kernel, dim3(grid), dim3(256), 0, s, up);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    up.col = p.cols[p.agg_a];
    up.col_b = p.cols[p.agg_b];
    hipLaunchKernelGGL(unfused_agg_kernel, dim3(grid), dim3(256), 0, s, up);
    return hipGetLastError();
}

struct HandoffParams {
    uint8_t* flags;
    uint32_t* gid;
    FusedParams p;
};
static_assert(sizeof(HandoffParams) <= 4096, "kernel arguments must fit the 4 KB kernarg segment");

// The whole query in one kernel, one row per thread, but with every hand-off
// between operators a store to and a later load from the per-row flag and
// group-id arrays in global memory (volatile, so none is kept in registers).
__global__ void __launch_bounds__(256) handoff_kernel(HandoffParams kernel_args) {
    (void)kernel_args;
    const HandoffParams& hp = *(const HandoffParams*)__builtin_amdgcn_kernarg_segment_ptr();
    const FusedParams& p = hp.p;
    volatile uint8_t* flags = hp.flags;
    volatile uint32_t* gid = hp.gid;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < p.n; i += stride) {
        flags[i] = 1u;
        gid[i] = 0u;
        for (int st = 0; st < p.nstages; ++st) {
            if (!flags[i]) break;
            const StageDev& S = p.st[st];
            uint32_t c;
            if (!device_stage_row(S, p.cols[S.col][i], c)) flags[i] = 0u;
            else if (S.gk_mode != GK_NONE) gid[i] = gid[i] + stage_gid_part(S, c);
        }
        if (!flags[i]) continue;
        const long long v = row_value(p.agg_kind, p.cols[p.agg_a][i], p.cols[p.agg_b][i]);
        const uint32_t g = gid[i];
        atomicAdd(&p.sums[g], (unsigned long long)v);
        atomicAdd(&p.counts[g], 1ull);
    }
}

hipError_t launch_handoff(const FusedParams& p, uint8_t* flags, uint32_t* gid, hipStream_t s) {
    if (p.n == 0) return hipSuccess;
    HandoffParams hp;
    memset(&hp, 0, sizeof hp);
    hp.flags = flags;
    hp.gid = gid;
    hp.p = p;
    hipLaunchKernelGGL(handoff_kernel, dim3(unfused_grid(p.n)), dim3(256), 0, s, hp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// streaming read of fact columns: the bandwidth the fused pass is compared with
// ---------------------------------------------------------------------------

// Adds every int32 of n_cols columns of n rows into *out (mod 2^64), reading
// the columns four at a time with 128-bit non-temporal loads, two 4-row
// items per lane: the fused kernel's load shape without any of its work.
__global__ void __launch_bounds__(512) read_columns_kernel(ReadParams kernel_args) {
    (void)kernel_args;
    const ReadParams& p = *(const ReadParams*)__builtin_amdgcn_kernarg_segment_ptr();
    const int64_t n_items = p.n / 4;
    const int64_t tile = (int64_t)blockDim.x * 2;
    unsigned long long acc = 0;
    for (int64_t base = (int64_t)blockIdx.x * tile; base < n_items; base += (int64_t)gridDim.x * tile) {
        for (int c0 = 0; c0 < p.n_cols; c0 += 4) {
            v4i x[4][2];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int64_t it = base + (int64_t)j * blockDim.x + threadIdx.x;
                    x[k][j] = v4i{0, 0, 0, 0};
                    if (c0 + k < p.n_cols && it < n_items)
                        x[k][j] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p.cols[c0 + k]) + it);
                }
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc += (unsigned long long)((long long)x[k][j].x + x[k][j].y + x[k][j].z + x[k][j].w);
        }
    }
    if (blockIdx.x == 0) {   // the last n mod 4 rows
        const int64_t r = n_items * 4 + (int64_t)threadIdx.x;
        if (r < p.n)
            for (int c = 0; c < p.n_cols; ++c) acc += (unsigned long long)(long long)p.cols[c][r];
    }
    acc = wave_sum_u64(acc);
    if ((threadIdx.x & 63u) == 0u) atomicAdd(p.out, acc);
}

hipError_t launch_read_columns(const ReadParams& p, int grid, hipStream_t s) {
    hipError_t e = launch_fill_u64(p.out, 1, s);
    if (e != hipSuccess || p.n == 0 || p.n_cols == 0) return e;
    hipLaunchKernelGGL(read_columns_kernel, dim3(grid), dim3(512), 0, s, p);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// partitioned aggregation: scan, scatter by partition, LDS aggregation
// ---------------------------------------------------------------------------

// One block: exclusive scan of the partition counts into part_start, and of
// the per-partition work items into chunk_start.
__global__ void __launch_bounds__(1024) part_scan_kernel(PartParams pp) {
    __shared__ uint32_t buf_r[1024], buf_c[1024];
    __shared__ uint32_t carry_r, carry_c;
    if (threadIdx.x == 0) {
        carry_r = 0u;
        carry_c = 0u;
    }
    __syncthreads();
    for (uint32_t base = 0; base < pp.n_parts; base += 1024u) {
        const uint32_t i = base + threadIdx.x;
        const uint32_t vr = i < pp.n_parts ? pp.part_count[i] : 0u;
        const uint32_t per = pp.skew_rows && vr > pp.skew_over ? pp.skew_rows : pp.chunk_rows;
        const uint32_t vc = vr / per + (vr % per != 0u ? 1u : 0u);
        buf_r[threadIdx.x] = vr;
        buf_c[threadIdx.x] = vc;
        __syncthreads();
        for (uint32_t off = 1; off < 1024u; off <<= 1) {
            const uint32_t ar = threadIdx.x >= off ? buf_r[threadIdx.x - off] : 0u;
            const uint32_t ac = threadIdx.x >= off ? buf_c[threadIdx.x - off] : 0u;
            __syncthreads();
            buf_r[threadIdx.x] += ar;
            buf_c[threadIdx.x] += ac;
            __syncthreads();
        }
        if (i < pp.n_parts) {
            pp.part_start[i] = carry_r + buf_r[threadIdx.x] - vr;
            pp.chunk_start[i] = carry_c + buf_c[threadIdx.x] - vc;
        }
        __syncthreads();
        if (threadIdx.x == 1023) {
            carry_r += buf_r[1023];
            carry_c += buf_c[1023];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        pp.part_start[pp.n_parts] = carry_r;
        pp.chunk_start[pp.n_parts] = carry_c;
    }
}

// Exclusive scan of n values by a 256-thread block: out[i] = carry + sum of
// in[0..i). in and out may be the same array (each thread reads its own run
// before writing it). Every thread must call it; returns the sum of in[0..n).
__device__ uint32_t block_scan_256(const uint32_t* in, uint32_t* out, uint32_t n, uint32_t carry,
                                   uint32_t* wtmp) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t per = (n + 255u) / 256u;
    const uint32_t b0 = threadIdx.x * per;
    uint32_t loc = 0;
    for (uint32_t k = 0; k < per; ++k)
        if (b0 + k < n) loc += in[b0 + k];
    uint32_t x = loc;
    for (uint32_t off = 1; off < 64u; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63u) wtmp[wave] = x;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (uint32_t w = 0; w < 4u; ++w) {
        const uint32_t t = wtmp[w];
        if (w < wave) before += t;
        total += t;
    }
    uint32_t run = carry + before + x - loc;
    for (uint32_t k = 0; k < per; ++k)
        if (b0 + k < n) {
            const uint32_t v = in[b0 + k];
            out[b0 + k] = run;
            run += v;
        }
    __syncthreads();
    return total;
}

// One block per partition q: the fused kernel's per-block counts of q become
// exclusive offsets within q (in place); their sum is q's record count.
__global__ void __launch_bounds__(256) part_offsets_kernel(PartParams pp) {
    __shared__ uint32_t wtmp[4];
    uint32_t* h = pp.part_hist + (uint64_t)blockIdx.x * pp.n_regions;
    uint32_t carry = 0;
    for (uint32_t b0 = 0; b0 < pp.n_regions; b0 += 4096u) {
        const uint32_t n = min(4096u, pp.n_regions - b0);
        carry += block_scan_256(h + b0, h + b0, n, carry, wtmp);
    }
    if (threadIdx.x == 0) {
        pp.part_count[blockIdx.x] = carry;
        if (pp.over && carry > pp.max_part) *pp.over = 1u;
    }
}

// One block per fused-kernel region: the region's records, kScatterChunk at a
// time, are counting-sorted by partition in LDS and written out so that each
// partition's records of the chunk form one contiguous run.
template <typename VT>
__global__ void __launch_bounds__(256) part_scatter_kernel(PartParams pp) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ uint32_t wtmp[4];
    constexpr int PER = kScatterChunk / 256;
    const uint32_t P = pp.n_parts;
    const int shift = pp.part_shift;
    VT* sval = reinterpret_cast<VT*>(smem);
    uint32_t* sgid = reinterpret_cast<uint32_t*>(sval + kScatterChunk);
    uint32_t* lcnt = sgid + kScatterChunk;
    uint32_t* lstart = lcnt + P;
    uint32_t* lcur = lstart + P;
    const uint32_t b = blockIdx.x;
    for (uint32_t q = threadIdx.x; q < P; q += blockDim.x) {
        lcur[q] = pp.part_start[q] + pp.part_hist[(uint64_t)q * pp.n_regions + b];
        lcnt[q] = 0u;
    }
    __syncthreads();
    const uint32_t n = pp.region_count[b];
    const uint32_t* rg = pp.rec_gid + (uint64_t)b * pp.part_cap;
    const VT* rv = static_cast<const VT*>(pp.rec_val) + (uint64_t)b * pp.part_cap;
    VT* out_val = static_cast<VT*>(pp.sorted_val);
    for (uint32_t c0 = 0; c0 < n; c0 += (uint32_t)kScatterChunk) {
        const uint32_t cn = min((uint32_t)kScatterChunk, n - c0);
        uint32_t g[PER], rk[PER];
        VT v[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t i = (uint32_t)k * 256u + threadIdx.x;
            g[k] = 0u;
            v[k] = 0;
            rk[k] = 0u;
            if (i < cn) {
                g[k] = rg[c0 + i];
                v[k] = rv[c0 + i];
            }
        }
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if ((uint32_t)k * 256u + threadIdx.x < cn) rk[k] = atomicAdd(&lcnt[g[k] >> shift], 1u);
        __syncthreads();
        block_scan_256(lcnt, lstart, P, 0u, wtmp);
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if ((uint32_t)k * 256u + threadIdx.x < cn) {
                const uint32_t pos = lstart[g[k] >> shift] + rk[k];
                sgid[pos] = g[k];
                sval[pos] = v[k];
            }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < cn; i += blockDim.x) {
            const uint32_t gi = sgid[i];
            const uint32_t q = gi >> shift;
            const uint32_t dest = lcur[q] + (i - lstart[q]);
            pp.sorted_gid[dest] = gi;
            out_val[dest] = sval[i];
        }
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < P; q += blockDim.x) {
            lcur[q] += lcnt[q];
            lcnt[q] = 0u;
        }
        __syncthreads();
    }
}

size_t part_scatter_lds_bytes(uint32_t n_parts, bool wide) {
    return (size_t)kScatterChunk * (wide ? 12u : 8u) + (size_t)n_parts * 12u;
}

// Work item c covers up to kPartChunk records of one partition q: sum them in
// an LDS table of q's groups. A partition with one work item adds its table
// straight into the outputs; otherwise each item stores its table as a partial
// that part_merge_kernel adds up. Either way each output group has exactly one
// writer in this pass, so plain read-add-write suffices (the outputs already
// hold what the fused kernel added for records past a region's capacity).
constexpr int kAggUnroll = 8;
constexpr int kAggBlock = 1024;   // one work item is summed by 16 waves sharing its LDS table

template <typename VT>
__global__ void __launch_bounds__(kAggBlock) part_agg_kernel(PartParams pp) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const uint32_t gpp = 1u << pp.part_shift;
    unsigned long long* lsum = reinterpret_cast<unsigned long long*>(smem);
    uint32_t* lcnt = reinterpret_cast<uint32_t*>(lsum + gpp);
    const uint32_t* sg = pp.sorted_gid;
    const VT* sv = static_cast<const VT*>(pp.sorted_val);
    const uint32_t n_items = pp.chunk_start[pp.n_parts];
    for (uint32_t c = blockIdx.x; c < n_items; c += gridDim.x) {
        // partition holding work item c: last q with chunk_start[q] <= c
        uint32_t lo = 0, hi = pp.n_parts;
        while (hi - lo > 1u) {
            const uint32_t mid = (lo + hi) >> 1;
            if (pp.chunk_start[mid] <= c) lo = mid;
            else hi = mid;
        }
        const uint32_t q = lo;
        const uint32_t r0 = pp.part_start[q] + (c - pp.chunk_start[q]) * (uint32_t)kPartChunk;
        const uint32_t r1 = min(r0 + (uint32_t)kPartChunk, pp.part_start[q + 1]);
        for (uint32_t k = threadIdx.x; k < gpp; k += blockDim.x) {
            lsum[k] = 0ull;
            lcnt[k] = 0u;
        }
        __syncthreads();
        const uint32_t g0 = q << pp.part_shift;
        // kAggUnroll records per thread in flight per step
        for (uint32_t i0 = r0; i0 < r1; i0 += kAggUnroll * blockDim.x) {
            uint32_t k[kAggUnroll];
            VT v[kAggUnroll];
#pragma unroll
            for (int u = 0; u < kAggUnroll; ++u) {
                const uint32_t i = i0 + (uint32_t)u * blockDim.x + threadIdx.x;
                k[u] = 0xFFFFFFFFu;
                v[u] = 0;
                if (i < r1) {
                    k[u] = sg[i] - g0;
                    v[u] = sv[i];
                }
            }
#pragma unroll
            for (int u = 0; u < kAggUnroll; ++u) {
                if (k[u] != 0xFFFFFFFFu) {
                    atomicAdd(&lsum[k[u]], (unsigned long long)(long long)v[u]);
                    atomicAdd(&lcnt[k[u]], 1u);
                }
            }
        }
        __syncthreads();
        const bool single = pp.chunk_start[q + 1] - pp.chunk_start[q] == 1u;
        const uint32_t kend = (uint32_t)min((uint64_t)gpp, pp.n_groups - g0);
        if (single) {
            for (uint32_t k = threadIdx.x; k < kend; k += blockDim.x) {
                pp.sums[g0 + k] += lsum[k];
                pp.counts[g0 + k] += lcnt[k];
            }
        } else {
            for (uint32_t k = threadIdx.x; k < kend; k += blockDim.x) {
                pp.item_sum[(uint64_t)c * gpp + k] = lsum[k];
                pp.item_cnt[(uint64_t)c * gpp + k] = lcnt[k];
            }
        }
        __syncthreads();
    }
}

// Groups of partitions with several work items: add the items' partials.
__global__ void __launch_bounds__(256) part_merge_kernel(PartParams pp) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t gpp = 1u << pp.part_shift;
    for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < pp.n_groups; g += stride) {
        const uint32_t q = (uint32_t)(g >> pp.part_shift);
        const uint32_t k = (uint32_t)g & (gpp - 1u);
        const uint32_t c0 = pp.chunk_start[q], c1 = pp.chunk_start[q + 1];
        if (c1 - c0 < 2u) continue;
        unsigned long long s = 0;
        unsigned long long n = 0;
        for (uint32_t c = c0; c < c1; ++c) {
            s += pp.item_sum[(uint64_t)c * gpp + k];
            n += pp.item_cnt[(uint64_t)c * gpp + k];
        }
        pp.sums[g] += s;
        pp.counts[g] += n;
    }
}

hipError_t launch_part_passes(const PartParams& pp, hipStream_t s) {
    hipLaunchKernelGGL(part_offsets_kernel, dim3(pp.n_parts), dim3(256), 0, s, pp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(part_scan_kernel, dim3(1), dim3(1024), 0, s, pp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const bool wide = pp.rec_wide != 0;
    const size_t agg_lds = (size_t)12u << pp.part_shift;
    if (wide) {
        hipLaunchKernelGGL(part_scatter_kernel<long long>, dim3(pp.n_regions), dim3(256),
                           part_scatter_lds_bytes(pp.n_parts, true), s, pp);
    } else {
        hipLaunchKernelGGL(part_scatter_kernel<int32_t>, dim3(pp.n_regions), dim3(256),
                           part_scatter_lds_bytes(pp.n_parts, false), s, pp);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (wide) hipLaunchKernelGGL(part_agg_kernel<long long>, dim3(512), dim3(kAggBlock), agg_lds, s, pp);
    else hipLaunchKernelGGL(part_agg_kernel<int32_t>, dim3(512), dim3(kAggBlock), agg_lds, s, pp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(part_merge_kernel, dim3(fill_grid(pp.n_groups)), dim3(256), 0, s, pp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// sliced hash probe: fact rows partitioned by the top bits of the key's hash
// ---------------------------------------------------------------------------

// Partition of key k: the top `bits` bits of its 32-bit multiplicative hash,
// which are also the top bits of its home slot in a table of at least 2^bits
// slots, so partition q probes only slice q of the table (and the slots
// that linear probing runs into past its end).
__device__ __forceinline__ uint32_t slice_of(int32_t k, int bits) {
    return ((uint32_t)k * 0x9E3779B1u) >> (32 - bits);
}

// Rows r .. r + 3 of a column (r a multiple of 4, the column 16-byte
// aligned): one 128-bit load, or row by row below r1 in a last partial group.
__device__ __forceinline__ void slice_load4(const int32_t* col, int64_t r, int64_t r1, int32_t* x) {
    if (r + 3 < r1) {
        const v4i v = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(col + r));
        x[0] = v.x;
        x[1] = v.y;
        x[2] = v.z;
        x[3] = v.w;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j] = r + j < r1 ? __builtin_nontemporal_load(col + r + j) : 0;
    }
}

// A thread's rows of the chunk at c0: kSliceRowsPerThread / 4 groups of 4,
// group i at c0 + 4 * (i * kSliceBlock + threadIdx.x). Which of them lie below
// r1 and pass every fact predicate, and their keys (0 for the others).
template <int RPT>
__device__ __forceinline__ void slice_load_keys(const SliceParams& sp, int64_t c0, int64_t r1, int32_t (&k)[RPT],
                                                bool (&ok)[RPT]) {
    constexpr int G = RPT / 4;
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const int64_t r = c0 + 4 * ((int64_t)i * kSliceBlock + threadIdx.x);
#pragma unroll
        for (int j = 0; j < 4; ++j) ok[4 * i + j] = r + j < r1;
    }
    for (int pi = 0; pi < sp.n_preds; ++pi) {
        const int32_t* col = sp.cols[sp.pred_col[pi]];
        const RangeTest t = sp.pred[pi];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int64_t r = c0 + 4 * ((int64_t)i * kSliceBlock + threadIdx.x);
            if (!(ok[4 * i] || ok[4 * i + 1] || ok[4 * i + 2] || ok[4 * i + 3])) continue;
            int32_t x[4];
            slice_load4(col, r, r1, x);
#pragma unroll
            for (int j = 0; j < 4; ++j) ok[4 * i + j] = ok[4 * i + j] && range_pass(t, x[j]);
        }
    }
    const int32_t* key = sp.cols[sp.key_col];
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const int64_t r = c0 + 4 * ((int64_t)i * kSliceBlock + threadIdx.x);
        int32_t x[4] = {0, 0, 0, 0};
        if (ok[4 * i] || ok[4 * i + 1] || ok[4 * i + 2] || ok[4 * i + 3]) slice_load4(key, r, r1, x);
#pragma unroll
        for (int j = 0; j < 4; ++j) k[4 * i + j] = ok[4 * i + j] ? x[j] : 0;
    }
}

// The pre-filter of the count pass: drops the rows whose key the table's
// pass filter rejects, and records for each of the thread's 4-row groups
// below r1 which of its rows stay (bit j: row 4 g + j), for the scatter pass.
template <int RPT>
__device__ __forceinline__ void slice_prefilter(const SliceParams& sp, int64_t c0, int64_t r1, const int32_t (&k)[RPT],
                                                bool (&ok)[RPT]) {
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        uint32_t w, m;
        if (ok[i]) ok[i] = filter_slot(sp.filt_kind, sp.filt_bits, sp.filt_key_min, k[i], w, m) &&
                           (sp.filt[w] & m) == m;
    }
#pragma unroll
    for (int i = 0; i < RPT / 4; ++i) {
        const int64_t r = c0 + 4 * ((int64_t)i * kSliceBlock + threadIdx.x);
        if (r < r1)
            sp.keep[r >> 2] = (uint8_t)((ok[4 * i] ? 1u : 0u) | (ok[4 * i + 1] ? 2u : 0u) | (ok[4 * i + 2] ? 4u : 0u) |
                                        (ok[4 * i + 3] ? 8u : 0u));
    }
}

// The scatter pass's rows after a pre-filter: which of the thread's rows the
// count pass kept, and their keys (0 for the others).
template <int RPT>
__device__ __forceinline__ void slice_load_kept(const SliceParams& sp, int64_t c0, int64_t r1, int32_t (&k)[RPT],
                                                bool (&ok)[RPT]) {
    const int32_t* key = sp.cols[sp.key_col];
#pragma unroll
    for (int i = 0; i < RPT / 4; ++i) {
        const int64_t r = c0 + 4 * ((int64_t)i * kSliceBlock + threadIdx.x);
        const uint32_t kb = r < r1 ? sp.keep[r >> 2] : 0u;
        int32_t x[4] = {0, 0, 0, 0};
        if (kb) slice_load4(key, r, r1, x);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            ok[4 * i + j] = ((kb >> j) & 1u) != 0u;
            k[4 * i + j] = ok[4 * i + j] ? x[j] : 0;
        }
    }
}

// Count pass: block b's passing rows per partition, into hist[q * grid + b].
// Lanes count into four interleaved copies of the histogram (by lane mod 4),
// so fewer lanes of one LDS atomic instruction hit the same counter.
__global__ void __launch_bounds__(kSliceBlock) slice_count_kernel(SliceParams sp) {
    __shared__ uint32_t lh[4 << SDB_MAX_SLICE_BITS];
    const uint32_t P = 1u << sp.bits;
    for (uint32_t q = threadIdx.x; q < 4u * P; q += blockDim.x) lh[q] = 0u;
    __syncthreads();
    uint32_t* mine = lh + (threadIdx.x & 3u);
    const int64_t r0 = (int64_t)blockIdx.x * sp.rows_per_block;
    const int64_t r1 = min(sp.n, r0 + sp.rows_per_block);
    for (int64_t c0 = r0; c0 < r1; c0 += kSliceChunk) {
        int32_t k[kSliceRowsPerThread];
        bool ok[kSliceRowsPerThread];
        slice_load_keys<kSliceRowsPerThread>(sp, c0, r1, k, ok);
        if (sp.filt) slice_prefilter<kSliceRowsPerThread>(sp, c0, r1, k, ok);
#pragma unroll
        for (int i = 0; i < kSliceRowsPerThread; ++i)
            if (ok[i]) atomicAdd(&mine[4u * slice_of(k[i], sp.bits)], 1u);
    }
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < P; q += blockDim.x)
        sp.hist[(uint64_t)q * gridDim.x + blockIdx.x] = lh[4u * q] + lh[4u * q + 1u] + lh[4u * q + 2u] + lh[4u * q + 3u];
}

// Exclusive scan of n values by the whole block (blockDim.x a multiple of
// 64, at most 1024): out[i] = carry + sum of in[0..i); in and out distinct.
// Every thread must call it; returns the sum of in[0..n).
__device__ uint32_t block_scan_any(const uint32_t* in, uint32_t* out, uint32_t n, uint32_t carry,
                                   uint32_t* wtmp) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const uint32_t per = (n + blockDim.x - 1u) / blockDim.x;
    const uint32_t b0 = threadIdx.x * per;
    uint32_t loc = 0;
    for (uint32_t k = 0; k < per; ++k)
        if (b0 + k < n) loc += in[b0 + k];
    uint32_t x = loc;
    for (uint32_t off = 1; off < 64u; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63u) wtmp[wave] = x;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (uint32_t w = 0; w < nw; ++w) {
        const uint32_t t = wtmp[w];
        if (w < wave) before += t;
        total += t;
    }
    uint32_t run = carry + before + x - loc;
    for (uint32_t k = 0; k < per; ++k)
        if (b0 + k < n) {
            out[b0 + k] = run;
            run += in[b0 + k];
        }
    __syncthreads();
    return total;
}

// Scatter pass: block b reads its rows again, RPT * kSliceBlock at a time,
// sorts each chunk's passing rows by partition in LDS (counting sort) and
// writes every partition's run of keys and values (TWO: both operands of a
// two-column aggregate, in chunks half as long so they fit LDS) after the ones
// block b wrote before (hist holds block b's first offset within each
// partition). With a pre-filter the passing rows are the ones the count pass
// kept, read from its per-group bytes instead of testing the predicates again.
template <int RPT, bool TWO>
__global__ void __launch_bounds__(kSliceBlock) slice_scatter_kernel(SliceParams sp) {
    constexpr int CHUNK = RPT * kSliceBlock;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ uint32_t wtmp[kSliceBlock / 64];
    int32_t* skey = reinterpret_cast<int32_t*>(smem);
    int32_t* sval = skey + CHUNK;
    int32_t* sval2 = sval + CHUNK;            // TWO only
    const uint32_t P = 1u << sp.bits;
    uint32_t* lcnt = reinterpret_cast<uint32_t*>(sval + (TWO ? 2 : 1) * CHUNK);
    uint32_t* lstart = lcnt + P;
    uint32_t* lcur = lstart + P;
    for (uint32_t q = threadIdx.x; q < P; q += blockDim.x) {
        lcur[q] = sp.part_start[q] + sp.hist[(uint64_t)q * gridDim.x + blockIdx.x];
        lcnt[q] = 0u;
    }
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * sp.rows_per_block;
    const int64_t r1 = min(sp.n, r0 + sp.rows_per_block);
    const int32_t* val = sp.cols[sp.val_col];
    const int32_t* val2 = sp.cols[TWO ? sp.val2_col : sp.val_col];
    for (int64_t c0 = r0; c0 < r1; c0 += CHUNK) {
        int32_t k[RPT], v[RPT], v2[RPT];
        bool ok[RPT];
        uint32_t rk[RPT];
        if (sp.keep) slice_load_kept<RPT>(sp, c0, r1, k, ok);
        else slice_load_keys<RPT>(sp, c0, r1, k, ok);
#pragma unroll
        for (int i = 0; i < RPT / 4; ++i) {
            const int64_t r = c0 + 4 * ((int64_t)i * kSliceBlock + threadIdx.x);
            int32_t x[4] = {0, 0, 0, 0}, y[4] = {0, 0, 0, 0};
            const bool any = ok[4 * i] || ok[4 * i + 1] || ok[4 * i + 2] || ok[4 * i + 3];
            if (any) slice_load4(val, r, r1, x);
            if (TWO && any) slice_load4(val2, r, r1, y);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v[4 * i + j] = x[j];
                v2[4 * i + j] = y[j];
            }
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            rk[i] = 0u;
            if (ok[i]) rk[i] = atomicAdd(&lcnt[slice_of(k[i], sp.bits)], 1u);
        }
        __syncthreads();
        const uint32_t cn = block_scan_any(lcnt, lstart, P, 0u, wtmp);
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (ok[i]) {
                const uint32_t pos = lstart[slice_of(k[i], sp.bits)] + rk[i];
                skey[pos] = k[i];
                sval[pos] = v[i];
                if (TWO) sval2[pos] = v2[i];
            }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < cn; i += blockDim.x) {
            const int32_t key = skey[i];
            const uint32_t q = slice_of(key, sp.bits);
            const uint64_t dest = (uint64_t)lcur[q] + (i - lstart[q]);
            if (dest < (uint64_t)sp.n) {   // always: both passes count the same rows
                sp.out_key[dest] = key;
                sp.out_val[dest] = sval[i];
                if (TWO) sp.out_val2[dest] = sval2[i];
            }
        }
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < P; q += blockDim.x) {
            lcur[q] += lcnt[q];
            lcnt[q] = 0u;
        }
        __syncthreads();
    }
}

// Rows 4 * t .. 4 * t + 3 of the n rows at col (16-byte aligned): one 128-bit
// load, or row by row in a last partial group (0 past its end).
__device__ __forceinline__ v4i slice_load_group(const int32_t* col, uint32_t t, uint32_t n) {
    v4i x = {0, 0, 0, 0};
    if (4u * t + 3u < n) {
        x = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(col) + t);
    } else {
        if (4u * t < n) x.x = __builtin_nontemporal_load(col + 4u * t);
        if (4u * t + 1u < n) x.y = __builtin_nontemporal_load(col + 4u * t + 1u);
        if (4u * t + 2u < n) x.z = __builtin_nontemporal_load(col + 4u * t + 2u);
    }
    return x;
}

// A thread's G groups of four rows (group i at row 4 * (i * kSliceBlock +
// threadIdx.x)) of the n rows at col; groups without a live row may be left out.
template <int G>
__device__ __forceinline__ void slice_load_values(const int32_t* col, uint32_t n, uint32_t live, int32_t (&v)[4 * G]) {
    if (n == 4u * G * kSliceBlock) {   // a whole chunk: no checks
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const v4i x =
                __builtin_nontemporal_load(reinterpret_cast<const v4i*>(col) + ((uint32_t)i * kSliceBlock + threadIdx.x));
            v[4 * i] = x.x;
            v[4 * i + 1] = x.y;
            v[4 * i + 2] = x.z;
            v[4 * i + 3] = x.w;
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
        v4i x = {0, 0, 0, 0};
        if ((live >> (4 * i)) & 0xFu) x = slice_load_group(col, (uint32_t)i * kSliceBlock + threadIdx.x, n);
        v[4 * i] = x.x;
        v[4 * i + 1] = x.y;
        v[4 * i + 2] = x.z;
        v[4 * i + 3] = x.w;
    }
}

// A thread's rows of the chunk of n rows at c0 (at most 4 * G * kSliceBlock):
// G groups of four, group i at row 4 * (i * kSliceBlock + threadIdx.x). Their
// keys, and in the result's bits which of them are below n and pass every fact
// predicate.
template <int G>
__device__ __forceinline__ uint32_t slice_load_live(const SliceParams& sp, int64_t c0, uint32_t n, int32_t (&k)[4 * G]) {
    uint32_t live = 0u;
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const uint32_t r = 4u * ((uint32_t)i * kSliceBlock + threadIdx.x);
        const uint32_t left = n > r ? min(n - r, 4u) : 0u;
        live |= ((1u << left) - 1u) << (4 * i);
    }
    for (int pi = 0; pi < sp.n_preds; ++pi) {
        const int32_t* col = sp.cols[sp.pred_col[pi]] + c0;
        const RangeTest t = sp.pred[pi];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if (!((live >> (4 * i)) & 0xFu)) continue;
            const v4i x = slice_load_group(col, (uint32_t)i * kSliceBlock + threadIdx.x, n);
            const uint32_t ok = (range_pass(t, x.x) ? 1u : 0u) | (range_pass(t, x.y) ? 2u : 0u) |
                                (range_pass(t, x.z) ? 4u : 0u) | (range_pass(t, x.w) ? 8u : 0u);
            live &= ~((ok ^ 0xFu) << (4 * i));
        }
    }
    slice_load_values<G>(sp.cols[sp.key_col] + c0, n, live, k);
    return live;
}

// Count pass of the LDS route (slice_count_kernel's counts), the next chunk's
// loads issued before this one is counted. Bound by the read of the columns.
__global__ void __launch_bounds__(kSliceBlock) slice_count_rec_kernel(SliceParams sp) {
    constexpr int G = 4;
    constexpr int64_t CHUNK = 4 * G * kSliceBlock;
    __shared__ uint32_t lh[4 << kSliceMaxBits];
    const uint32_t P = 1u << sp.bits;
    for (uint32_t q = threadIdx.x; q < 4u * P; q += kSliceBlock) lh[q] = 0u;
    __syncthreads();
    uint32_t* mine = lh + (threadIdx.x & 3u);
    const int64_t r0 = (int64_t)blockIdx.x * sp.rows_per_block;
    const int64_t r1 = min(sp.n, r0 + sp.rows_per_block);
    int32_t k[4 * G], next[4 * G];
    uint32_t live = 0u, next_live = 0u;
    if (r0 < r1) live = slice_load_live<G>(sp, r0, (uint32_t)min(r1 - r0, CHUNK), k);
    for (int64_t c0 = r0; c0 < r1; c0 += CHUNK) {
        if (c0 + CHUNK < r1)
            next_live = slice_load_live<G>(sp, c0 + CHUNK, (uint32_t)min(r1 - c0 - CHUNK, CHUNK), next);
#pragma unroll
        for (int i = 0; i < 4 * G; ++i)
            if ((live >> i) & 1u) atomicAdd(&mine[4u * slice_of(k[i], sp.bits)], 1u);
#pragma unroll
        for (int i = 0; i < 4 * G; ++i) k[i] = next[i];
        live = next_live;
    }
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < P; q += kSliceBlock)
        sp.hist[(uint64_t)q * gridDim.x + blockIdx.x] = lh[4u * q] + lh[4u * q + 1u] + lh[4u * q + 2u] + lh[4u * q + 3u];
}

// Writes the n rows of an LDS window that starts at place w0 of its chunk.
template <bool TWO>
__device__ __forceinline__ void slice_write_window(const SliceParams& sp, const unsigned long long* srec,
                                                   const int32_t* sval2, const uint32_t* lcur, uint32_t w0, uint32_t n) {
    for (uint32_t i = threadIdx.x; i < n; i += kSliceBlock) {
        const unsigned long long rec = srec[i];
        const uint32_t dest = lcur[slice_of((int32_t)(uint32_t)rec, sp.bits)] + w0 + i;
        if ((int64_t)dest < sp.n) {   // always: both passes count the same rows
            sp.out_rec[dest] = rec;
            if constexpr (TWO) sp.out_val2[dest] = sval2[i];
        }
    }
}

// Scatter pass of the LDS route, whose partitions are many (up to 2,048): the
// longer the chunk a block sorts at a time, the longer the runs it writes, so
// a chunk's rows (4 * G a thread) stay in registers and only WINDOW of them
// at a time pass through LDS in partition order. Bound by the runs' partial
// lines. The next chunk's loads are issued before the last window is written.
// `load(at, n, k, v, v2)` reads a thread's rows of the n at row `at` and
// returns which of them are there.
template <int G, bool TWO, class Load>
__device__ __forceinline__ void slice_scatter_rows(const SliceParams& sp, const Load& load_rows) {
    constexpr int RPT = 4 * G, CHUNK = RPT * kSliceBlock;
    constexpr uint32_t WINDOW = TWO ? 8192u : 16384u;
    static_assert(CHUNK <= 65536, "16-bit places in a chunk");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ uint32_t wtmp[kSliceBlock / 64];
    unsigned long long* srec = reinterpret_cast<unsigned long long*>(smem);
    int32_t* sval2 = reinterpret_cast<int32_t*>(srec + WINDOW);   // TWO only
    const uint32_t P = 1u << sp.bits;
    uint32_t* lcnt = reinterpret_cast<uint32_t*>(sval2 + (TWO ? WINDOW : 0u));
    uint32_t* lstart = lcnt + P;
    uint32_t* lcur = lstart + P;      // next position in the partition, less lstart once that is known
    for (uint32_t q = threadIdx.x; q < P; q += kSliceBlock) {
        lcur[q] = sp.part_start[q] + sp.hist[(uint64_t)q * gridDim.x + blockIdx.x];
        lcnt[q] = 0u;
    }
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * sp.rows_per_block;
    const int64_t r1 = min(sp.n, r0 + sp.rows_per_block);
    int32_t k[RPT], v[RPT], v2[TWO ? RPT : 4];
    uint32_t live = 0u;
    const auto load = [&](int64_t at) { live = load_rows(at, (uint32_t)min(r1 - at, (int64_t)CHUNK), k, v, v2); };
    if (r0 < r1) load(r0);
    for (int64_t c0 = r0; c0 < r1; c0 += CHUNK) {
        // each row's rank in its partition, then its place in partition order, two to a register
        uint32_t place[RPT / 2];
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            uint32_t r = 0u;
            if ((live >> i) & 1u) r = atomicAdd(&lcnt[slice_of(k[i], sp.bits)], 1u);
            place[i / 2] = (i & 1) ? place[i / 2] | (r << 16) : r;
            if (G > 4 && i % 8 == 7) __builtin_amdgcn_sched_barrier(0);   // at most 8 results in registers
        }
        // (the partitions are worked out again below rather than kept in registers)
#pragma unroll
        for (int i = 0; i < (G > 4 ? RPT : 0); ++i) asm volatile("" : "+v"(k[i]));
        __syncthreads();
        const uint32_t cn = __builtin_amdgcn_readfirstlane(block_scan_any(lcnt, lstart, P, 0u, wtmp));
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const uint32_t s = lstart[slice_of(k[i], sp.bits)];
            place[i / 2] += (i & 1) ? s << 16 : s;
            if (G > 4 && i % 8 == 7) __builtin_amdgcn_sched_barrier(0);
        }
        for (uint32_t q = threadIdx.x; q < P; q += kSliceBlock) lcur[q] -= lstart[q];
        uint32_t w0 = 0u;
        for (;;) {
#pragma unroll
            for (int i = 0; i < RPT; ++i) {
                const uint32_t at = ((place[i / 2] >> ((i & 1) * 16)) & 0xFFFFu) - w0;
                if (((live >> i) & 1u) && at < WINDOW) {
                    srec[at] = ((unsigned long long)(uint32_t)v[i] << 32) | (uint32_t)k[i];
                    if constexpr (TWO) sval2[at] = v2[i];
                }
            }
            if (w0 + WINDOW >= cn) break;
            __syncthreads();
            slice_write_window<TWO>(sp, srec, sval2, lcur, w0, WINDOW);
            __syncthreads();
            w0 += WINDOW;
        }
        if (c0 + CHUNK < r1) load(c0 + CHUNK);
        __syncthreads();
        slice_write_window<TWO>(sp, srec, sval2, lcur, w0, cn - w0);
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < P; q += kSliceBlock) {
            lcur[q] += lstart[q] + lcnt[q];
            lcnt[q] = 0u;
        }
        __syncthreads();
    }
}

template <int G, bool TWO>
__global__ void __launch_bounds__(kSliceBlock) slice_scatter_rec_kernel(SliceParams sp) {
    slice_scatter_rows<G, TWO>(sp, [&](int64_t at, uint32_t n, int32_t (&k)[4 * G], int32_t (&v)[4 * G], auto& v2) {
        const uint32_t live = slice_load_live<G>(sp, at, n, k);
        slice_load_values<G>(sp.cols[sp.val_col] + at, n, live, v);
        if constexpr (TWO) slice_load_values<G>(sp.cols[sp.val2_col] + at, n, live, v2);
        return live;
    });
}

size_t slice_scatter_rec_lds_bytes(uint32_t n_parts, bool two) {
    return (two ? 8192u * 12u : 16384u * 8u) + (size_t)n_parts * 12u;
}

// The tile order of the fused launch over the partitioned rows. Loop index t
// runs on block t mod grid, which the dispatcher places on XCD t mod 8 (the
// grids here are multiples of 8); giving XCD x only the tiles whose first row
// lies in a partition q with q mod 8 == x means each XCD's L2 holds the table
// slices of its own partitions, and each slice is probed by one XCD's 32 CUs
// for eight times as long, so the blocks drift apart by fewer slices.
// One thread: the rank of each partition's first tile among its XCD's tiles.
__global__ void slice_tile_base_kernel(SliceParams sp) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    const uint32_t P = 1u << sp.bits;
    const uint64_t T = (uint64_t)sp.tile_rows;
    uint64_t run[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (uint32_t q = 0; q < P; ++q) {
        const uint64_t a = ((uint64_t)sp.part_start[q] + T - 1) / T;
        const uint64_t b = ((uint64_t)sp.part_start[q + 1] + T - 1) / T;
        sp.tile_base[q] = (uint32_t)run[q & 7u];
        run[q & 7u] += b - a;
    }
}

// One thread per tile j (first row j * tile_rows below the passing-row count):
// its partition q (binary search of the partition starts), then its slot
// 8 * rank + (q mod 8) in the map (filled with -1 before).
__global__ void __launch_bounds__(256) slice_tile_map_kernel(SliceParams sp) {
    const uint32_t P = 1u << sp.bits;
    const uint64_t T = (uint64_t)sp.tile_rows;
    const uint64_t total = sp.part_start[P];
    const uint64_t n_phys = (total + T - 1) / T;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n_phys; j += stride) {
        const uint64_t row = j * T;
        uint32_t lo = 0, hi = P;   // last partition whose start is <= row
        while (hi - lo > 1u) {
            const uint32_t mid = (lo + hi) >> 1;
            if ((uint64_t)sp.part_start[mid] <= row) lo = mid;
            else hi = mid;
        }
        const uint64_t first = ((uint64_t)sp.part_start[lo] + T - 1) / T;
        const uint64_t v = 8u * ((uint64_t)sp.tile_base[lo] + (j - first)) + (lo & 7u);
        if (v < (uint64_t)sp.n_vtiles) sp.tile_map[v] = (int32_t)j;
    }
}

// rows per thread of the scatter chunk: half as many with two value columns
constexpr int kSliceRowsPerThreadTwo = kSliceRowsPerThread / 2;

size_t slice_scatter_lds_bytes(uint32_t n_parts, bool two) {
    const size_t chunk = (size_t)kSliceBlock * (two ? kSliceRowsPerThreadTwo : kSliceRowsPerThread);
    return chunk * 4u * (two ? 3u : 2u) + (size_t)n_parts * 12u;
}

hipError_t launch_slice_partition(const SliceParams& sp, int grid, hipStream_t s) {
    if (sp.bits < 1 || sp.bits > kSliceMaxBits || grid < 1) return hipErrorInvalidValue;
    const uint32_t P = 1u << sp.bits;
    if (!sp.out_rec && sp.bits > SDB_MAX_SLICE_BITS) return hipErrorInvalidValue;
    if (sp.out_rec) hipLaunchKernelGGL(slice_count_rec_kernel, dim3(grid), dim3(kSliceBlock), 0, s, sp);
    else hipLaunchKernelGGL(slice_count_kernel, dim3(grid), dim3(kSliceBlock), 0, s, sp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    PartParams pp;
    std::memset(&pp, 0, sizeof pp);
    pp.n_parts = P;
    pp.n_regions = (uint32_t)grid;
    pp.part_hist = sp.hist;
    pp.part_count = sp.part_count;
    pp.part_start = sp.part_start;
    pp.chunk_start = sp.chunk_start;
    pp.chunk_rows = sp.out_rec ? sp.item_rows : (uint32_t)kPartChunk;
    pp.skew_rows = sp.out_rec ? sp.skew_rows : 0u;
    pp.skew_over = sp.skew_over;
    hipLaunchKernelGGL(part_offsets_kernel, dim3(P), dim3(256), 0, s, pp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(part_scan_kernel, dim3(1), dim3(1024), 0, s, pp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const bool two = sp.val2_col >= 0;
    if (sp.out_rec && two)
        hipLaunchKernelGGL((slice_scatter_rec_kernel<4, true>), dim3(grid), dim3(kSliceBlock),
                           slice_scatter_rec_lds_bytes(P, true), s, sp);
    // chunks of 32,768 rows where 16,384 would leave runs of at most 8 rows and a
    // block has many chunks (2,048 partitions: 600M rows 3.67 against 4.18 ms, but
    // 40M rows in 256 partitions 190 against 134 us)
    else if (sp.out_rec && sp.bits >= 11 && sp.rows_per_block >= 16 * 32768)
        hipLaunchKernelGGL((slice_scatter_rec_kernel<8, false>), dim3(grid), dim3(kSliceBlock),
                           slice_scatter_rec_lds_bytes(P, false), s, sp);
    else if (sp.out_rec)
        hipLaunchKernelGGL((slice_scatter_rec_kernel<4, false>), dim3(grid), dim3(kSliceBlock),
                           slice_scatter_rec_lds_bytes(P, false), s, sp);
    else if (two)
        hipLaunchKernelGGL((slice_scatter_kernel<kSliceRowsPerThreadTwo, true>), dim3(grid), dim3(kSliceBlock),
                           slice_scatter_lds_bytes(P, true), s, sp);
    else
        hipLaunchKernelGGL((slice_scatter_kernel<kSliceRowsPerThread, false>), dim3(grid), dim3(kSliceBlock),
                           slice_scatter_lds_bytes(P, false), s, sp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (sp.tile_map) {
        e = launch_fill_u32(reinterpret_cast<uint32_t*>(sp.tile_map), (uint64_t)sp.n_vtiles, 0xFFFFFFFFu, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(slice_tile_base_kernel, dim3(1), dim3(64), 0, s, sp);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        const uint64_t phys = (uint64_t)sp.n_vtiles / 8u;
        const int g = (int)std::min<uint64_t>(1024u, std::max<uint64_t>(1u, (phys + 255u) / 256u));
        hipLaunchKernelGGL(slice_tile_map_kernel, dim3(g), dim3(256), 0, s, sp);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// the LDS route of the sliced hash probe
// ---------------------------------------------------------------------------

constexpr uint32_t kAggHashes = 1u << kSliceAggHashBits;
constexpr uint32_t kAggFree = 0xFFFFu;   // hash value without an entry
static_assert(kSliceAggEntries < kAggFree, "16-bit entry numbers");

// The LDS table of a slice's passing keys: kAggHashes 16-bit entry numbers,
// looked up from the hash bits below the slice's with linear probing (at most
// 4,608 of 32,768 are taken, so most rows end at the first), and the entries.
struct SliceTable {
    uint16_t* at;              // kAggHashes entry numbers or kAggFree
    uint32_t* key;             // kSliceAggEntries each
    uint16_t* slot;            // where the key stands: table slots from the slice's (or round's) first on
    uint32_t* rows;
    unsigned long long* sum;
};

__device__ __forceinline__ uint32_t slice_hash(uint32_t key, int bits) {
    return ((key * 0x9E3779B1u) << bits) >> (32 - kSliceAggHashBits);
}

// The entry of `key`, or kAggFree, from hash value h on.
__device__ __forceinline__ uint32_t slice_find(const SliceTable& t, uint32_t key, uint32_t h) {
    uint32_t e = t.at[h];
    while (e != kAggFree && t.key[e] != key) {
        h = (h + 1u) & (kAggHashes - 1u);
        e = t.at[h];
    }
    return e;
}

// A table slot read for slice q: whether it holds a passing row of the slice.
__device__ __forceinline__ bool slice_slot_passes(unsigned long long slot, uint32_t q, int bits) {
    const uint32_t enc = (uint32_t)(slot >> 32);
    return enc != 0u && enc != 0xFFFFFFFFu && slice_of((int32_t)(uint32_t)slot, bits) == q;
}

// Puts the wave's slots that hold a passing row of slice q into the LDS table
// (as slot number `at`), as long as entries are free; *n counts them all. The
// whole wave calls it together.
__device__ __forceinline__ void slice_put(unsigned long long slot, uint32_t at, uint32_t q, int bits,
                                          const SliceTable& t, uint32_t* n) {
    const bool pass = slice_slot_passes(slot, q, bits);
    const uint32_t lane = threadIdx.x & 63u;
    const unsigned long long m = __ballot(pass);
    uint32_t e = 0;
    if (lane == 0 && m) e = atomicAdd(n, (uint32_t)__popcll(m));
    e = __shfl(e, 0, 64) + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    if (pass && e < kSliceAggEntries) {
        const uint32_t key = (uint32_t)slot;
        t.key[e] = key;
        t.slot[e] = (uint16_t)at;
        t.rows[e] = 0u;
        t.sum[e] = 0ull;
        // the first free hash value from the key's on takes the entry
        uint32_t* words = reinterpret_cast<uint32_t*>(t.at);
        uint32_t h = slice_hash(key, bits);
        uint32_t old = words[h >> 1];
        for (;;) {
            const uint32_t sh = (h & 1u) * 16u;
            if (((old >> sh) & 0xFFFFu) != kAggFree) {
                h = (h + 1u) & (kAggHashes - 1u);
                old = words[h >> 1];
                continue;
            }
            const uint32_t got = atomicCAS(&words[h >> 1], old, (old & ~(0xFFFFu << sh)) | (e << sh));
            if (got == old) break;
            old = got;
        }
    }
}

// Puts the passing rows among table slots [lo, hi), counted from the slice's
// first, into the LDS table. The whole block calls it together.
__device__ __forceinline__ void slice_fill_table(const SliceAggParams& ap, uint32_t q, uint32_t lo, uint32_t hi,
                                                 const SliceTable& t, uint32_t* n) {
    constexpr int U = 16;
    const unsigned long long* tab = static_cast<const unsigned long long*>(ap.st.map);
    const uint32_t base = q * (ap.st.nslots >> ap.bits);
    for (uint32_t i0 = lo; i0 < hi; i0 += U * blockDim.x) {
        unsigned long long slot[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = i0 + (uint32_t)u * blockDim.x + threadIdx.x;
            slot[u] = i < hi ? tab[(base + i) & ap.st.hmask] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            slice_put(slot[u], i0 + (uint32_t)u * blockDim.x + threadIdx.x - lo, q, ap.bits, t, n);
    }
}

// Adds rows [r0, r1) of a partition to the entries of their keys. A thread
// takes kAggPairs pairs of rows a step (16-byte loads), the next step's loads
// issued before this one's lookups; the first lookups of its rows are made
// together, and the rows that met another key go on one by one.
constexpr int kAggPairs = 3;
// Atomics of one address are performed one after the other, so where a wave
// holds at least kAggSame rows of its first row's key it adds them up itself.
constexpr int kAggSame = 32;

// The sum over the wave, in lane 63: shifts within the rows of 16 lanes, then
// the rows' last lanes to the rows after them. (Through LDS, as __shfl_xor
// does, the sums would cost what the atomics do.)
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_add_u64(unsigned long long v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xF, true);
    return v + (((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ unsigned long long wave_last_sum_u64(unsigned long long v) {
    v = dpp_add_u64<0x111, 0xF>(v);   // row_shr:1
    v = dpp_add_u64<0x112, 0xF>(v);
    v = dpp_add_u64<0x114, 0xF>(v);
    v = dpp_add_u64<0x118, 0xF>(v);
    v = dpp_add_u64<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add_u64<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}

template <bool TWO>
__device__ __forceinline__ void slice_load_pairs(const unsigned long long* rec, const int32_t* rec_b, uint32_t at,
                                                 uint32_t n, u64x2 (&x)[kAggPairs], unsigned long long (&w)[kAggPairs]) {
#pragma unroll
    for (int k = 0; k < kAggPairs; ++k) {
        uint32_t i = at + 2u * ((uint32_t)k * 1024u + threadIdx.x);
        i = i < n ? i : 0u;   // past the last row: any pair of the item
        x[k] = __builtin_nontemporal_load(reinterpret_cast<const u64x2*>(rec + i));
        if (TWO) w[k] = __builtin_nontemporal_load(reinterpret_cast<const unsigned long long*>(rec_b + i));
    }
}

template <bool TWO>
__device__ __forceinline__ void slice_add_rows(const SliceAggParams& ap, uint32_t r0, uint32_t r1,
                                               const SliceTable& t) {
    constexpr int U = 2 * kAggPairs;
    constexpr uint32_t kStep = U * 1024u;
    if (r0 >= r1) return;
    const uint32_t skip = r0 & 1u;   // pairs start at even rows
    const uint32_t n = r1 - r0 + skip;
    const unsigned long long* rec = ap.rec + (r0 - skip);
    const int32_t* rec_b = TWO ? ap.rec_b + (r0 - skip) : nullptr;
    u64x2 x[kAggPairs];
    unsigned long long w[kAggPairs];
    slice_load_pairs<TWO>(rec, rec_b, 0u, n, x, w);
    for (uint32_t at = 0; at < n; at += kStep) {
        uint32_t key[U], h[U], e[U], k[U];
        const bool full = at >= skip && at + kStep <= n;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            key[u] = (uint32_t)((u & 1) ? x[u >> 1].y : x[u >> 1].x);
            h[u] = slice_hash(key[u], ap.bits);
            e[u] = t.at[h[u]];
        }
        long long v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned long long r = (u & 1) ? x[u >> 1].y : x[u >> 1].x;
            v[u] = (long long)(int32_t)(uint32_t)(r >> 32);
            if (TWO) {
                const long long y = (long long)(int32_t)(uint32_t)((u & 1) ? w[u >> 1] >> 32 : w[u >> 1]);
                v[u] = ap.agg_kind == SDB_AGG_MUL ? v[u] * y : (ap.agg_kind == SDB_AGG_SUB ? v[u] - y : v[u] + y);
            }
        }
        if (at + kStep < n) slice_load_pairs<TWO>(rec, rec_b, at + kStep, n, x, w);
        if (!full) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = at + 2u * ((uint32_t)(u >> 1) * 1024u + threadIdx.x) + (u & 1);
                if (i < skip || i >= n) e[u] = kAggFree;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = t.key[e[u] != kAggFree ? e[u] : 0u];
        // many rows of one key (looked for in the first of the step's rows only)
        const uint32_t lead_key = (uint32_t)__builtin_amdgcn_readfirstlane((int)key[0]);
        const bool many = __popcll(__ballot(key[0] == lead_key)) >= kAggSame;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (e[u] != kAggFree && k[u] != key[u]) e[u] = slice_find(t, key[u], (h[u] + 1u) & (kAggHashes - 1u));
            if (many) {
                const uint32_t lead = (uint32_t)__builtin_amdgcn_readfirstlane((int)e[u]);
                const unsigned long long same = __ballot(e[u] == lead);
                if (lead != kAggFree && __popcll(same) >= kAggSame) {
                    const unsigned long long sum = wave_last_sum_u64(e[u] == lead ? (unsigned long long)v[u] : 0ull);
                    if ((threadIdx.x & 63u) == 63u) {
                        atomicAdd(&t.rows[lead], (uint32_t)__popcll(same));
                        atomicAdd(&t.sum[lead], sum);
                    }
                    if (e[u] == lead) e[u] = kAggFree;
                }
            }
            if (e[u] != kAggFree) {
                atomicAdd(&t.rows[e[u]], 1u);
                atomicAdd(&t.sum[e[u]], (unsigned long long)v[u]);
            }
        }
    }
}

__device__ __forceinline__ void slice_clear_table(const SliceTable& t) {
    v4u* w = reinterpret_cast<v4u*>(t.at);
    for (uint32_t k = threadIdx.x; k < kAggHashes / 8u; k += blockDim.x) w[k] = v4u{~0u, ~0u, ~0u, ~0u};
}

__device__ __forceinline__ unsigned long long* xcd_copy(const SliceAggParams& ap) {
    return ap.xcd_copies > 0 ? ap.xtab + 2ull * ap.n_groups * (xcc_id() & (uint32_t)(ap.xcd_copies - 1)) : nullptr;
}

// Adds a sum over `rows` rows to group g of the outputs, or of this XCD's copy.
__device__ __forceinline__ void add_group_total(const SliceAggParams& ap, unsigned long long* xt, uint32_t g,
                                                unsigned long long sum, unsigned long long rows) {
    atomicAdd(xt ? &xt[2ull * g] : &ap.sums[g], sum);
    atomicAdd(xt ? &xt[2ull * g + 1u] : &ap.counts[g], rows);
}

// Sums the partitioned rows by dimension row before the join: a work item (at
// most kSliceAggItem rows of partition q) loads the passing rows of table
// slice q into an LDS table, adds every row's value and count to its key's
// entry (rows whose key is not there die: misses and filtered rows alike), and
// then adds each entry once to its group. A passing key's rows so cost two LDS
// atomics each and its group one update per work item, instead of a record
// (or an atomic) per row. With few groups (lds_groups) the block keeps them in
// LDS and flushes them once; with more, the entries leave as records by range
// of groups (what is past a range's capacity, and the rest, with global
// atomics).
// Keys of a slice stand between its first slot and the first empty slot past
// its end (linear probing), so that is the range of slots read. Should more
// than kSliceAggEntries of them pass (keys that hash unevenly), the rows are
// gone through once for every kSliceAggEntries slots.
template <bool TWO>
__global__ void __launch_bounds__(1024) slice_agg_kernel(SliceAggParams kernel_args) {
    (void)kernel_args;
    const SliceAggParams& ap = *(const SliceAggParams*)__builtin_amdgcn_kernarg_segment_ptr();
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    __shared__ uint32_t s_len, s_n, s_q;
    __shared__ uint32_t s_emit[kSliceEmitMaxRanges], s_emit_at[kSliceEmitMaxRanges];
    for (uint32_t r = threadIdx.x; r < kSliceEmitMaxRanges; r += blockDim.x) s_emit[r] = 0u;
    SliceTable t;
    t.sum = reinterpret_cast<unsigned long long*>(smem);
    t.at = reinterpret_cast<uint16_t*>(t.sum + kSliceAggEntries);
    t.key = reinterpret_cast<uint32_t*>(t.at + kAggHashes);
    t.rows = t.key + kSliceAggEntries;
    t.slot = reinterpret_cast<uint16_t*>(t.rows + kSliceAggEntries);
    unsigned long long* gsum = reinterpret_cast<unsigned long long*>(t.slot + kSliceAggEntries);
    uint32_t* gcnt = reinterpret_cast<uint32_t*>(gsum + ap.lds_groups);
    const StageDev& S = ap.st;
    const unsigned long long* tab = static_cast<const unsigned long long*>(S.map);
    const uint32_t P = 1u << ap.bits, per = S.nslots >> ap.bits;
    for (uint32_t g = threadIdx.x; g < ap.lds_groups; g += blockDim.x) {
        gsum[g] = 0ull;
        gcnt[g] = 0u;
    }
    unsigned long long* xt = xcd_copy(ap);
    const uint32_t n_items = ap.chunk_start[P];
    for (uint32_t c = blockIdx.x; c < n_items; c += gridDim.x) {
        // partition holding work item c
        for (uint32_t i = threadIdx.x; i < P; i += blockDim.x)
            if (ap.chunk_start[i] <= c && c < ap.chunk_start[i + 1]) s_q = i;
        if (threadIdx.x == 0) s_n = 0u;
        slice_clear_table(t);
        __syncthreads();
        const uint32_t q = __builtin_amdgcn_readfirstlane(s_q);
        const uint32_t base = q * per;
        slice_fill_table(ap, q, 0u, per, t, &s_n);
        if (threadIdx.x < 64u) {
            // the slots past the slice's up to the first empty one
            for (uint32_t off = per;; off += 64u) {
                const uint32_t i = off + threadIdx.x;
                const unsigned long long slot = i < S.nslots ? tab[(base + i) & S.hmask] : 0ull;
                const unsigned long long m = __ballot((slot >> 32) == 0ull);
                const uint32_t end = m ? (uint32_t)__ffsll((long long)m) - 1u : 64u;
                slice_put(threadIdx.x < end ? slot : 0ull, i, q, ap.bits, t, &s_n);
                if (m) {
                    if (threadIdx.x == 0) s_len = off + end;
                    break;
                }
            }
        }
        __syncthreads();
        const uint32_t len = __builtin_amdgcn_readfirstlane(s_len);
        const uint32_t n_pass = __builtin_amdgcn_readfirstlane(s_n);
        // one round over the rows when the slice's entries fit the table and
        // their slot numbers 16 bits, else one for every kSliceAggEntries slots
        const bool one = n_pass <= kSliceAggEntries && len <= 65536u;
        const bool none = n_pass == 0u;
        // the partition's rows in equal shares over its work items
        const uint32_t p0 = ap.part_start[q], p1 = ap.part_start[q + 1];
        const uint32_t c0 = ap.chunk_start[q], share = (p1 - p0 - 1u) / (ap.chunk_start[q + 1] - c0) + 1u;
        const uint32_t r0 = p0 + min((c - c0) * share, p1 - p0);
        const uint32_t r1 = min(p1 - r0, share) + r0;
        for (uint32_t lo = 0; lo < len && !none;) {
            const uint32_t hi = one ? len : min(len, lo + kSliceAggEntries);
            if (!one) {
                __syncthreads();
                slice_clear_table(t);
                if (threadIdx.x == 0) s_n = 0u;
                __syncthreads();
                slice_fill_table(ap, q, lo, hi, t, &s_n);
                __syncthreads();
            }
            const uint32_t n_entries = one ? n_pass : __builtin_amdgcn_readfirstlane(s_n);
            slice_add_rows<TWO>(ap, r0, r1, t);
            __syncthreads();
            // every entry once into its group; its code from the table slot
            constexpr int E = (int)((kSliceAggEntries + 1023u) / 1024u);
            {
                uint32_t g[E], rows[E], rank[E];
                unsigned long long sum[E];
#pragma unroll
                for (int u = 0; u < E; ++u) {
                    const uint32_t e = (uint32_t)u * 1024u + threadIdx.x;
                    rows[u] = e < n_entries ? t.rows[e] : 0u;
                    g[u] = 0u;
                    if (rows[u]) g[u] = (uint32_t)(tab[(base + lo + t.slot[e]) & S.hmask] >> 32) - 1u;
                }
#pragma unroll
                for (int u = 0; u < E; ++u) {
                    if (!rows[u]) continue;
                    sum[u] = t.sum[(uint32_t)u * 1024u + threadIdx.x];
                    g[u] = S.gk_mode == GK_ONE ? g[u] * S.gk_stride[0]
                         : S.gk_mode == GK_GENERAL ? code_contribution(S, g[u]) : 0u;
                }
                if (ap.emit_ranges) {
                    // ranks within the ranges, one claim per range for the block's entries
#pragma unroll
                    for (int u = 0; u < E; ++u)
                        if (rows[u]) rank[u] = atomicAdd(&s_emit[g[u] >> kSliceEmitShift], 1u);
                    __syncthreads();
                    for (uint32_t r = threadIdx.x; r < ap.emit_ranges; r += blockDim.x) {
                        const uint32_t n = s_emit[r];
                        s_emit[r] = 0u;
                        s_emit_at[r] = n ? atomicAdd(&ap.emit_fill[r], n) : 0u;
                    }
                    __syncthreads();
                }
#pragma unroll
                for (int u = 0; u < E; ++u) {
                    if (!rows[u]) continue;
                    if (ap.lds_groups) {
                        atomicAdd(&gsum[g[u]], sum[u]);
                        atomicAdd(&gcnt[g[u]], rows[u]);
                        continue;
                    }
                    if (ap.emit_ranges) {
                        const uint32_t r = g[u] >> kSliceEmitShift;
                        const uint32_t at = s_emit_at[r] + rank[u];
                        if (at < ap.emit_cap) {
                            const v4u rec = {g[u], rows[u], (uint32_t)sum[u], (uint32_t)(sum[u] >> 32)};
                            reinterpret_cast<v4u*>(ap.emit)[(uint64_t)r * ap.emit_cap + at] = rec;
                            continue;
                        }
                    }
                    add_group_total(ap, xt, g[u], sum[u], rows[u]);
                }
            }
            lo = hi;
        }
        __syncthreads();
    }
    __syncthreads();
    for (uint32_t g = threadIdx.x; g < ap.lds_groups; g += blockDim.x)
        if (gcnt[g]) {
            atomicAdd(&ap.sums[g], gsum[g]);
            atomicAdd(&ap.counts[g], (unsigned long long)gcnt[g]);
        }
}

// One block per kSliceEmitChunk records of a range of groups (block
// x: chunk, y: range): sums them in LDS, then adds the chunk's groups.
__global__ void __launch_bounds__(1024) slice_merge_kernel(SliceAggParams kernel_args) {
    (void)kernel_args;
    const SliceAggParams& ap = *(const SliceAggParams*)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr uint32_t G = 1u << kSliceEmitShift;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned long long* lsum = reinterpret_cast<unsigned long long*>(smem);
    unsigned long long* lrows = lsum + G;
    const uint32_t r = blockIdx.y, n = min(ap.emit_fill[r], ap.emit_cap);
    const uint32_t i0 = blockIdx.x * kSliceEmitChunk;
    if (i0 >= n) return;
    const uint32_t i1 = min(n - i0, kSliceEmitChunk) + i0, g0 = r << kSliceEmitShift;
    for (uint32_t k = threadIdx.x; k < 2u * G; k += blockDim.x) lsum[k] = 0ull;
    __syncthreads();
    const v4u* rec = reinterpret_cast<const v4u*>(ap.emit) + (uint64_t)r * ap.emit_cap;
    constexpr int U = 8;
    for (uint32_t j0 = i0; j0 < i1; j0 += U * blockDim.x) {
        v4u x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = j0 + (uint32_t)u * blockDim.x + threadIdx.x;
            x[u] = i < i1 ? __builtin_nontemporal_load(rec + i) : v4u{g0, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (x[u].y) {
                atomicAdd(&lsum[x[u].x - g0], ((unsigned long long)x[u].w << 32) | x[u].z);
                atomicAdd(&lrows[x[u].x - g0], (unsigned long long)x[u].y);
            }
    }
    __syncthreads();
    unsigned long long* xt = xcd_copy(ap);
    for (uint32_t k = threadIdx.x; k < G; k += blockDim.x)
        if (lrows[k]) add_group_total(ap, xt, g0 + k, lsum[k], lrows[k]);
}

hipError_t launch_slice_agg(const SliceAggParams& ap, int grid, hipStream_t s) {
    if (ap.bits < 1 || ap.bits > kSliceMaxBits || grid < 1 || ap.lds_groups > kSliceAggMaxGroups ||
        ap.emit_ranges > kSliceEmitMaxRanges)
        return hipErrorInvalidValue;
    const size_t lds = (size_t)kSliceAggEntries * 18u + (size_t)kAggHashes * 2u + (size_t)ap.lds_groups * 12u;
    if (ap.rec_b) hipLaunchKernelGGL(slice_agg_kernel<true>, dim3(grid), dim3(1024), lds, s, ap);
    else hipLaunchKernelGGL(slice_agg_kernel<false>, dim3(grid), dim3(1024), lds, s, ap);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !ap.emit_ranges) return e;
    const uint32_t chunks = (ap.emit_cap + kSliceEmitChunk - 1u) / kSliceEmitChunk;
    hipLaunchKernelGGL(slice_merge_kernel, dim3(chunks, ap.emit_ranges), dim3(1024),
                       (size_t)16u << kSliceEmitShift, s, ap);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// sliced build of a hash table
// ---------------------------------------------------------------------------

// Compare-and-swap inserts all over a table larger than the caches run at
// about 9G rows/s (8.4M rows into 2^24 slots: 978 us, and 20 us to fill them;
// this build 275 us, 183 of them the slices, whose Bloom filter bits are
// atomics bound for the memory side). Here the rows' slot values are first
// partitioned by table slice (the probe's own passes), each slice is built in
// LDS and written whole, and the few rows whose linear probing leaves their
// slice are inserted last; no slot is filled before.
__global__ void __launch_bounds__(kSliceBlock) hash_count_kernel(HashSliceParams hp) {
    __shared__ uint32_t lh[1 << kSliceMaxBits];
    const uint32_t P = 1u << hp.bits;
    for (uint32_t q = threadIdx.x; q < P; q += kSliceBlock) lh[q] = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *hp.spill_n = 0u;
        *hp.over = 0u;
    }
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * hp.rows_per_block;
    const int64_t r1 = min(hp.bp.n, r0 + hp.rows_per_block);
    constexpr int U = 16;
    for (int64_t i0 = r0 + threadIdx.x; i0 < r1; i0 += U * kSliceBlock) {
        int32_t k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) k[u] = i0 + u * kSliceBlock < r1 ? hp.bp.key[i0 + u * kSliceBlock] : 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kSliceBlock < r1) atomicAdd(&lh[slice_of(k[u], hp.bits)], 1u);
    }
    __syncthreads();
    for (uint32_t q = threadIdx.x; q < P; q += kSliceBlock) hp.hist[(uint64_t)q * gridDim.x + blockIdx.x] = lh[q];
}

__global__ void __launch_bounds__(kSliceBlock) hash_scatter_kernel(HashSliceParams hp) {
    // a slice with more rows than slots cannot be built: no pass does anything
    // from here on, and the host builds the table with inserts
    if (*hp.over) {
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&hp.bp.stats->dup, kHashSliceRetry);
        return;
    }
    SliceParams sp;
    sp.n = hp.bp.n;
    sp.rows_per_block = hp.rows_per_block;
    sp.bits = hp.bits;
    sp.hist = hp.hist;
    sp.part_start = hp.part_start;
    sp.out_rec = hp.rec;
    constexpr int G = 4;
    slice_scatter_rows<G, false>(sp, [&](int64_t at, uint32_t n, int32_t (&k)[4 * G], int32_t (&v)[4 * G], auto&) {
        uint32_t live = 0u, pass;
        int32_t x[4 * G];
        const BuildParams& bp = hp.bp;
        const auto column = [&](const int32_t* col, int32_t (&to)[4 * G], uint32_t which) {
#pragma unroll
            for (int u = 0; u < 4 * G; ++u)
                to[u] = (which >> u) & 1u ? col[at + (uint32_t)u * kSliceBlock + threadIdx.x] : 0;
        };
#pragma unroll
        for (int u = 0; u < 4 * G; ++u) live |= ((uint32_t)u * kSliceBlock + threadIdx.x < n ? 1u : 0u) << u;
        column(bp.key, k, live);
        pass = live;
        for (int q = 0; q < bp.n_preds; ++q) {
            column(bp.cols[bp.pred_col[q]], x, live);
#pragma unroll
            for (int u = 0; u < 4 * G; ++u)
                if (!range_pass(bp.pred[q], x[u])) pass &= ~(1u << u);
        }
#pragma unroll
        for (int u = 0; u < 4 * G; ++u) v[u] = 1;   // code + 1
        for (int p = 0; p < bp.n_payloads; ++p) {
            column(bp.cols[bp.payload_col[p]], x, pass);
#pragma unroll
            for (int u = 0; u < 4 * G; ++u)
                v[u] = (int32_t)((uint32_t)v[u] + ((uint32_t)x[u] - (uint32_t)bp.pmin[p]) * bp.pdiv[p]);
        }
#pragma unroll
        for (int u = 0; u < 4 * G; ++u)
            if (!((pass >> u) & 1u)) v[u] = -1;
        return live;
    });
}

// One block per slice.
__global__ void __launch_bounds__(1024) hash_slice_kernel(HashSliceParams hp) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned long long* slots = reinterpret_cast<unsigned long long*>(smem);
    const BuildParams& bp = hp.bp;
    const uint32_t q = blockIdx.x, per = (uint32_t)(bp.nslots >> hp.bits);
    const uint32_t r0 = hp.part_start[q], n = hp.part_start[q + 1] - r0;
    if (*hp.over) return;
    for (uint32_t i = threadIdx.x; i < per; i += 1024u) slots[i] = 0ull;
    __syncthreads();
    constexpr int U = 8;
    for (uint32_t i0 = threadIdx.x; i0 < n; i0 += U * 1024u) {
        unsigned long long rec[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            rec[u] = i0 + u * 1024u < n ? __builtin_nontemporal_load(hp.rec + r0 + (i0 + u * 1024u)) : 0ull;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (i0 + u * 1024u >= n) continue;
            hash_filter_key(bp, rec[u]);
            const uint32_t k = (uint32_t)rec[u];
            uint32_t h = ((k * 0x9E3779B1u) >> bp.hshift) & (per - 1u);
            for (;;) {
                const unsigned long long old = atomicCAS(&slots[h], 0ull, rec[u]);
                if (old == 0ull) break;
                if ((uint32_t)old == k) {
                    atomicOr(&bp.stats->dup, 1u);
                    break;
                }
                if (++h == per) {
                    const uint32_t at = atomicAdd(hp.spill_n, 1u);
                    if (at < hp.spill_cap) hp.spill[at] = rec[u];
                    else atomicOr(&bp.stats->dup, kHashSliceRetry);
                    break;
                }
            }
        }
    }
    __syncthreads();
    unsigned long long* tab = static_cast<unsigned long long*>(bp.map) + (uint64_t)q * per;
    for (uint32_t i = threadIdx.x; i < per; i += 1024u) tab[i] = slots[i];
}

// The rows past their slices' ends, once every slice is written. Not where the
// slices were given up: the table then holds what the workspace held, and
// probing it for an empty slot could walk all of it for every row.
__global__ void __launch_bounds__(256) hash_spill_kernel(HashSliceParams hp) {
    if (hp.bp.stats->dup & kHashSliceRetry) return;
    const uint32_t n = min(*hp.spill_n, hp.spill_cap);
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n; i += gridDim.x * 256u) hash_place(hp.bp, hp.spill[i]);
}

hipError_t launch_hash_slices(const HashSliceParams& hp, hipStream_t s) {
    const uint32_t P = 1u << hp.bits;
    if (hp.bits < 1 || hp.bits > kSliceMaxBits || (hp.bp.nslots >> hp.bits) > (1ull << kHashSliceSlotBits) ||
        (hp.bp.nslots >> hp.bits) < 1)
        return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    if (hp.bp.filt && !hp.bp.filt_via_bytes) {
        e = launch_fill_u32(hp.bp.filt, (hp.bp.filt_bits + 31) / 32, 0u, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(hash_count_kernel, dim3(kHashSliceGrid), dim3(kSliceBlock), 0, s, hp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    PartParams pp;
    std::memset(&pp, 0, sizeof pp);
    pp.n_parts = P;
    pp.n_regions = kHashSliceGrid;
    pp.part_hist = hp.hist;
    pp.part_count = hp.part_count;
    pp.part_start = hp.part_start;
    pp.chunk_start = hp.chunk_start;
    pp.chunk_rows = (uint32_t)kPartChunk;
    pp.over = hp.over;
    pp.max_part = (uint32_t)(hp.bp.nslots >> hp.bits);
    hipLaunchKernelGGL(part_offsets_kernel, dim3(P), dim3(256), 0, s, pp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(part_scan_kernel, dim3(1), dim3(1024), 0, s, pp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(hash_scatter_kernel, dim3(kHashSliceGrid), dim3(kSliceBlock),
                       slice_scatter_rec_lds_bytes(P, false), s, hp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(hash_slice_kernel, dim3(P), dim3(1024), (size_t)(hp.bp.nslots >> hp.bits) * 8u, s, hp);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(hash_spill_kernel, dim3(64), dim3(256), 0, s, hp);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// finalize: order-preserving compaction of the group table
// ---------------------------------------------------------------------------

__device__ __forceinline__ bool group_present(const FinalizeParams& fp, uint64_t g) {
    if (g >= fp.n_groups) return false;
    return fp.scalar ? true : fp.counts[g] > 0;
}

__global__ void __launch_bounds__(kFinBlock) fin_count_kernel(FinalizeParams fp) {
    __shared__ unsigned int wsum[kFinBlock / 64];
    const uint64_t base = (uint64_t)blockIdx.x * kFinGroupsPerBlock;
    unsigned int c = 0;
    for (int k = 0; k < kFinPerThread; ++k) c += group_present(fp, base + (uint64_t)k * kFinBlock + threadIdx.x);
    for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned int t = 0;
        for (int w = 0; w < kFinBlock / 64; ++w) t += wsum[w];
        fp.block_off[blockIdx.x] = t;
    }
}

// One block turns the per-block counts into exclusive offsets and writes the total.
__global__ void __launch_bounds__(1024) fin_scan_kernel(FinalizeParams fp) {
    __shared__ long long buf[1024];
    __shared__ long long carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t base = 0; base < fp.n_blocks; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const long long v = i < fp.n_blocks ? fp.block_off[i] : 0;
        buf[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {       // Hillis-Steele inclusive scan
            const long long add = threadIdx.x >= (unsigned)off ? buf[threadIdx.x - off] : 0;
            __syncthreads();
            buf[threadIdx.x] += add;
            __syncthreads();
        }
        const long long incl = buf[threadIdx.x];
        if (i < fp.n_blocks) fp.block_off[i] = carry + incl - v;
        __syncthreads();
        if (threadIdx.x == 1023) carry += incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) fp.out_n[0] = carry;
}

// Group g of the table goes to row o of the result.
__device__ __forceinline__ void fin_write(const FinalizeParams& fp, uint64_t g, uint64_t o) {
    for (int q = 0; q < fp.n_keys; ++q)
        fp.out_keys[o * fp.n_keys + q] = (int32_t)(((uint32_t)g / fp.stride[q]) % fp.radix[q]) + fp.key_min[q];
    fp.out_sums[o] = fp.sums[g];
    fp.out_counts[o] = fp.counts[g];
}

// `scanned`: block_off holds offsets (fin_scan_kernel); else the blocks'
// counts, and every block adds up those before its own (at most
// kFinMaxPrefix: 32 KB from L2, cheaper than a launch for the scan).
__global__ void __launch_bounds__(kFinBlock) fin_scatter_kernel(FinalizeParams fp, bool scanned) {
    __shared__ unsigned int wcnt[kFinBlock / 64];
    __shared__ long long run;
    __shared__ unsigned long long part[kFinBlock / 64];
    if (scanned) {
        if (threadIdx.x == 0) run = fp.block_off[blockIdx.x];
    } else {
        unsigned long long c = 0;
        for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kFinBlock) c += (unsigned long long)fp.block_off[i];
        c = wave_sum_u64(c);
        if ((threadIdx.x & 63u) == 0u) part[threadIdx.x >> 6] = c;
        __syncthreads();
        if (threadIdx.x == 0) {
            run = (long long)(part[0] + part[1] + part[2] + part[3]);
            if (blockIdx.x == gridDim.x - 1u) fp.out_n[0] = run + fp.block_off[blockIdx.x];
        }
    }
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kFinGroupsPerBlock;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int k = 0; k < kFinPerThread; ++k) {
        const uint64_t g = base + (uint64_t)k * kFinBlock + threadIdx.x;
        const bool present = group_present(fp, g);
        const unsigned long long m = __ballot(present);
        const unsigned int before_in_wave = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) wcnt[wave] = __popcll(m);
        __syncthreads();
        unsigned int before = before_in_wave;
        unsigned int total = 0;
        for (int w = 0; w < kFinBlock / 64; ++w) {
            if (w < wave) before += wcnt[w];
            total += wcnt[w];
        }
        if (present) fin_write(fp, g, (uint64_t)run + before);
        __syncthreads();
        if (threadIdx.x == 0) run += total;
        __syncthreads();
    }
}

// Up to kFinOneGroups groups by one block: thread t holds groups k * 1024 + t,
// whose counts it loads together; a group's place is the number of groups
// present before it, from the waves' ballots.
__global__ void __launch_bounds__(1024) fin_one_kernel(FinalizeParams fp) {
    constexpr int R = (int)(kFinOneGroups / 1024);
    __shared__ uint32_t cnt[R * 16];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const int rounds = (int)((fp.n_groups + 1023u) / 1024u);
    unsigned long long m[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        m[k] = 0ull;
        if (k < rounds) {
            m[k] = __ballot(group_present(fp, (uint64_t)k * 1024u + threadIdx.x));
            if (lane == 0) cnt[k * 16 + wave] = (uint32_t)__popcll(m[k]);
        }
    }
    __syncthreads();
    if (threadIdx.x < 64u) {   // exclusive scan of the (at most 128) wave counts by one wave, two a lane
        const uint32_t n = (uint32_t)rounds * 16u;
        const uint32_t a = 2u * lane < n ? cnt[2u * lane] : 0u, b = 2u * lane + 1u < n ? cnt[2u * lane + 1u] : 0u;
        uint32_t x = a + b;
        for (uint32_t off = 1; off < 64u; off <<= 1) {
            const uint32_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        if (2u * lane < n) cnt[2u * lane] = x - a - b;
        if (2u * lane + 1u < n) cnt[2u * lane + 1u] = x - b;
        if (lane == 63u) fp.out_n[0] = x;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R; ++k)
        if ((m[k] >> lane) & 1ull)
            fin_write(fp, (uint64_t)k * 1024u + threadIdx.x,
                      cnt[k * 16 + wave] + (uint32_t)__popcll(m[k] & ((1ull << lane) - 1ull)));
}

hipError_t launch_finalize(const FinalizeParams& fp, hipStream_t s) {
    if (fp.n_groups <= kFinOneGroups) {
        hipLaunchKernelGGL(fin_one_kernel, dim3(1), dim3(1024), 0, s, fp);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(fin_count_kernel, dim3((unsigned)fp.n_blocks), dim3(kFinBlock), 0, s, fp);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const bool scan = fp.n_blocks > kFinMaxPrefix;
    if (scan) {
        hipLaunchKernelGGL(fin_scan_kernel, dim3(1), dim3(1024), 0, s, fp);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fin_scatter_kernel, dim3((unsigned)fp.n_blocks), dim3(kFinBlock), 0, s, fp, scan);
    return hipGetLastError();
}

// ---- fixed device scratch for sdb_run_star_query_noalloc ------------------
//
// Callers that cannot allocate device memory (code under stream capture,
// serving loops, harnesses that forbid hipMalloc) run a query with this
// file-scope array as its run scratch. Every device the library runs on holds
// its own copy from the code object's load until the process ends. In host
// code the array's name is only a host-side stand-in: its device address comes
// from hipGetSymbolAddress, taken once per device with that device current.

static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

hipError_t noalloc_scratch(void** out) {
    static std::mutex mu;
    static void* per_device[kNoallocMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kNoallocMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!per_device[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p || ((uintptr_t)p & 255u) != 0) return hipErrorInvalidSymbol;
        per_device[dev] = p;
    }
    *out = per_device[dev];
    return hipSuccess;
}

}  // namespace sdb
