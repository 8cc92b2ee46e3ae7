// HyperLogLog sketches of the distinct k-mers of every bin, from the k-mer
// occurrences of its super-mers: the alternative the table-size estimate
// of Sec. 3.4.1 is compared with. The work items are chunks of kHllChunk
// super-mers of one bin, so a large bin is spread over many workgroups. A
// workgroup keeps the 2^p registers of its item's bin in LDS; a wave cuts 64
// super-mers into segments of about equal length, and each lane rolls the
// windows of a segment, hashes every canonical key and raises register (top p
// bits of the hash) to the rank of the first set bit of the remaining bits. The item's registers are then
// merged into the bin's with atomic maxima (the registers start at zero), so
// the result does not depend on how the bin was split.
//
// Bound by vector issue, some 95 lane instructions a window of 65 bases (two
// 64-bit multiplies of the hash take a third): 344 M windows in 0.95 ms. A
// super-mer per thread took 2.56 ms: its lengths differ, and a wave ran on for
// the longest of 64.
#include "../../include/gerbil.h"
#include "common.h"
#include "internal.h"

namespace gerbil {
namespace {

constexpr uint32_t kHllBlock = 256;
constexpr uint64_t kHllSeed = 0x5bd1e9955bd1e995ull;   // not the table seed: an independent hash

// Registers raised by one k-mer: its canonical key's hash, 64 bits.
template <int D>
__device__ __forceinline__ uint64_t hash_window(const uint32_t (&fw)[D], const uint32_t (&rc)[D], uint32_t canonical,
                                                uint32_t tail) {
    bool take = rc[0] < fw[0], same = rc[0] == fw[0];
    if (D > 1 && __ballot(same) != 0ull) {
#pragma unroll
        for (int i = 1; i < D; i++) {
            take = same ? rc[i] < fw[i] : take;
            same = same && rc[i] == fw[i];
        }
    }
    take = take && canonical;
    constexpr int W = (D + 1) / 2;
    uint64_t key[W];
#pragma unroll
    for (int i = 0; i < W; i++) {
        const uint32_t hi = take ? rc[2 * i] : fw[2 * i];
        const uint32_t lo = 2 * i + 1 < D ? (take ? rc[2 * i + 1 < D ? 2 * i + 1 : 0] : fw[2 * i + 1 < D ? 2 * i + 1 : 0]) : 0u;
        key[i] = ((uint64_t)hi << 32) | lo;
    }
    key[W - 1] >>= tail;
    return key_hash<W>(key, kHllSeed);
}

constexpr uint32_t kHllChunk = 2048;   // super-mers per work item
constexpr uint32_t kHllOwners = 256;   // segments a wave lists the super-mers of at a time

template <int D>
__global__ void __launch_bounds__(kHllBlock) k_hll(const uint64_t* __restrict__ packed, uint64_t n_bytes,
                                                   const uint64_t* __restrict__ desc,
                                                   const uint64_t* __restrict__ bin_off, uint32_t n_bins, uint32_t k,
                                                   uint32_t canonical, uint32_t p, uint32_t* __restrict__ regs) {
    constexpr uint32_t kSeg = D <= 6 ? 8 : 16;      // windows of a segment at most
    constexpr uint32_t kLoads = (D + 4) / 2;        // words that hold D + 1 half words from any base on
    __shared__ uint8_t owner[kHllBlock / 64][kHllOwners];
    extern __shared__ uint32_t lds[];
    const uint32_t m = 1u << p, tid = threadIdx.x, lane = __lane_id(), wave = uniform(tid >> 6);
    uint32_t* R = lds;              // [m] registers of the current item's bin
    uint32_t* pre = lds + m;        // [n_bins + 1] first work item of every bin
    uint32_t* part = pre + n_bins + 1;   // [kHllBlock] scan scratch
    // work items per bin and their prefix: thread t takes bins [t*per, (t+1)*per)
    const uint32_t per = (n_bins + kHllBlock - 1) / kHllBlock;
    uint32_t sum = 0;
    for (uint32_t e = 0; e < per; e++) {
        const uint32_t b = tid * per + e;
        if (b < n_bins) sum += (uint32_t)((bin_off[b + 1] - bin_off[b] + kHllChunk - 1) / kHllChunk);
    }
    part[tid] = sum;
    __syncthreads();
    for (uint32_t off = 1; off < kHllBlock; off <<= 1) {
        const uint32_t y = tid >= off ? part[tid - off] : 0u;
        __syncthreads();
        part[tid] += y;
        __syncthreads();
    }
    uint32_t run = tid ? part[tid - 1] : 0u;
    for (uint32_t e = 0; e < per; e++) {
        const uint32_t b = tid * per + e;
        if (b < n_bins) {
            pre[b] = run;
            run += (uint32_t)((bin_off[b + 1] - bin_off[b] + kHllChunk - 1) / kHllChunk);
        }
    }
    if (tid == kHllBlock - 1) pre[n_bins] = part[kHllBlock - 1];
    __syncthreads();
    const uint32_t total = pre[n_bins];
    const uint32_t pad = 32u * D - 2u * k;          // 0 .. 30 bits
    const uint32_t tail_mask = 0xFFFFFFFFu << pad;
    const uint32_t tail = 2 * (32u * ((D + 1) / 2) - k);
    const int64_t last = (int64_t)((n_bytes + 31) >> 5);   // two zero words follow the stream
    for (uint32_t item = blockIdx.x; item < total; item += gridDim.x) {
        uint32_t lo = 0, hi = n_bins;   // the bin of the item: last b with pre[b] <= item
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (pre[mid] <= item) lo = mid; else hi = mid;
        }
        const uint32_t b = lo;
        const uint64_t d0 = bin_off[b] + (uint64_t)(item - pre[b]) * kHllChunk;
        const uint64_t d1 = d0 + kHllChunk < bin_off[b + 1] ? d0 + kHllChunk : bin_off[b + 1];
        for (uint32_t j = tid; j < m; j += kHllBlock) R[j] = 0;
        __syncthreads();
        uint64_t dd = d0 + tid < d1 ? desc[d0 + tid] : 0ull;
        for (uint64_t d = d0 + wave * 64; d < d1; d += kHllBlock) {
            // this lane's super-mer, cut into segments of about equal length
            const uint64_t start = dd >> 24;
            uint32_t nk = (uint32_t)(dd & 0xFFFFFFu);
            if (nk == 0 || start + nk - 1 + k > n_bytes) nk = 0;   // never read out of range
            dd = d + kHllBlock + lane < d1 ? desc[d + kHllBlock + lane] : 0ull;
            const uint32_t ns = (nk + kSeg - 1) / kSeg;
            const uint32_t each = ns ? nk / ns : 0u, more = nk - each * ns;   // the first `more` have one more
            const uint32_t incl = wave_incl_sum(ns), first = incl - ns;
            const uint32_t total_segs = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            for (uint32_t y0 = 0; y0 < total_segs; y0 += 64) {
                if (y0 % kHllOwners == 0) {   // whose the next segments are
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    const uint32_t lo = first > y0 ? first - y0 : 0u;
                    const uint32_t hi = incl > y0 ? (incl - y0 < kHllOwners ? incl - y0 : kHllOwners) : 0u;
                    for (uint32_t i = lo; i < hi; i++) owner[wave][i] = (uint8_t)lane;
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                }
                const uint32_t y = y0 + lane;
                const int from = 4 * (int)owner[wave][y < total_segs ? y % kHllOwners : (total_segs - 1) % kHllOwners];
                const uint32_t s = y - (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)first);
                const uint32_t em = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(each | more << 6));
                const uint32_t len = y < total_segs ? (em & 63u) + (s < em >> 6 ? 1u : 0u) : 0u;
                const uint32_t off = s * (em & 63u) + (s < em >> 6 ? s : em >> 6);
                uint64_t pos = ((uint64_t)(uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(start >> 32)) << 32) |
                               (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)(uint32_t)start);
                pos = len ? pos + off : 0ull;
                // D + 1 words of 16 bases from base pos on: the first window and what follows it
                uint32_t x[D + 1];
                {
                    const int64_t e = ((int64_t)pos - 1) >> 5;   // (so that no funnel shift is by 32)
                    const uint32_t at = (uint32_t)(pos - 1) & 31u, sh = 30u - 2u * (at & 15u);
                    uint32_t h[2 * kLoads];
#pragma unroll
                    for (uint32_t i = 0; i < kLoads; i++) {
                        const int64_t q = e + (int64_t)i;
                        const uint64_t v = packed[q < last ? q : last];
                        h[2 * i] = (uint32_t)(v >> 32);   // a word's first 16 bases are its high half
                        h[2 * i + 1] = (uint32_t)v;
                    }
                    uint32_t a = at >= 16 ? h[1] : h[0];
#pragma unroll
                    for (int i = 0; i <= D; i++) {
                        const uint32_t b = at >= 16 ? h[i + 2] : h[i + 1];
                        x[i] = funnel(a, b, sh);
                        a = b;
                    }
                }
                uint32_t nx = funnel(x[D - 1], x[D], pad);   // the bases that follow the first window
                uint32_t fw[D], rc[D];
#pragma unroll
                for (int i = 0; i < D; i++) fw[i] = x[i];
                fw[D - 1] &= tail_mask;
                {
                    uint32_t z[D + 1];
#pragma unroll
                    for (int i = 0; i < D; i++) z[i] = revcomp16(fw[D - 1 - i]);
                    z[D] = 0;
#pragma unroll
                    for (int i = 0; i < D; i++) rc[i] = pad ? funnel(z[i], z[i + 1], 32u - pad) : z[i];
                    rc[D - 1] &= tail_mask;
                }
                const uint32_t most = wave_max(len);
                for (uint32_t i = 0;;) {
                    const uint64_t hash = hash_window<D>(fw, rc, canonical, tail);
                    const uint32_t hi = (uint32_t)(hash >> 32), lo = (uint32_t)hash;
                    const uint32_t idx = hi >> (32 - p), rest = funnel(hi, lo, 32 - p);
                    uint32_t rho = (uint32_t)__builtin_clz(rest | 1u) + 1u;
                    if (__ballot(rest <= 1u) != 0ull && rest <= 1u)   // (one hash in 2^31)
                        rho = rest ? 32u : 33u + (uint32_t)__builtin_clz((lo << p) | (1u << (p - 1)));
                    if (i < len) atomicMax(&R[idx], rho);
                    if (++i >= most) break;
                    const uint32_t b = nx >> 30;
                    nx <<= 2;
#pragma unroll
                    for (int q = 0; q + 1 < D; q++) fw[q] = funnel(fw[q], fw[q + 1], 30);
                    fw[D - 1] = (fw[D - 1] << 2) | (b << pad);
#pragma unroll
                    for (int q = D - 1; q > 0; q--) rc[q] = funnel(rc[q - 1], rc[q], 2);
                    rc[0] = (rc[0] >> 2) | ((3u - b) << 30);
                    rc[D - 1] &= tail_mask;
                }
            }
        }
        __syncthreads();
        for (uint32_t j = tid; j < m; j += kHllBlock)
            if (R[j]) atomicMax(&regs[((uint64_t)b << p) + j], R[j]);
        __syncthreads();   // R is cleared for the next item
    }
}

template <int D>
hipError_t hll_d(const uint64_t* packed, uint64_t n_bytes, const uint64_t* desc, const uint64_t* bin_off,
                 uint32_t n_bins, uint32_t k, uint32_t canonical, uint32_t p, uint32_t* regs, hipStream_t s) {
    const size_t lds = ((size_t)1 << p) * 4 + ((size_t)n_bins + 1) * 4 + (size_t)kHllBlock * 4;
    if (hipFuncSetAttribute((const void*)k_hll<D>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return hipErrorInvalidValue;
    hipError_t e = launch_fill_u32(regs, (uint64_t)n_bins << p, 0u, s);   // merged by atomic maxima
    if (e != hipSuccess) return e;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        cus = 1;
    // every item is taken by some workgroup (grid stride); as many as are resident
    uint32_t per_cu = 160u * 1024u / ((uint32_t)lds + kHllBlock / 64 * kHllOwners);
    per_cu = per_cu < 1 ? 1 : per_cu > 8 ? 8 : per_cu;
    const uint32_t grid = per_cu * (uint32_t)cus;
    hipLaunchKernelGGL(k_hll<D>, dim3(grid), dim3(kHllBlock), lds, s, packed, n_bytes, desc, bin_off, n_bins, k,
                       canonical, p, regs);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_hll(const uint64_t* packed, uint64_t n_bytes, const uint64_t* desc, const uint64_t* bin_off,
                      uint32_t n_bins, uint32_t k, uint32_t canonical, uint32_t p, uint32_t* regs, hipStream_t s) {
    switch ((k + 15) / 16) {
        case 1: return hll_d<1>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 2: return hll_d<2>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 3: return hll_d<3>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 4: return hll_d<4>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 5: return hll_d<5>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 6: return hll_d<6>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 7: return hll_d<7>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 8: return hll_d<8>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 9: return hll_d<9>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 10: return hll_d<10>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 11: return hll_d<11>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 12: return hll_d<12>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 13: return hll_d<13>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 14: return hll_d<14>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 15: return hll_d<15>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 16: return hll_d<16>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 17: return hll_d<17>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 18: return hll_d<18>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 19: return hll_d<19>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 20: return hll_d<20>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 21: return hll_d<21>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 22: return hll_d<22>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 23: return hll_d<23>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 24: return hll_d<24>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 25: return hll_d<25>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 26: return hll_d<26>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 27: return hll_d<27>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 28: return hll_d<28>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 29: return hll_d<29>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
        case 30: return hll_d<30>(packed, n_bytes, desc, bin_off, n_bins, k, canonical, p, regs, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace gerbil
