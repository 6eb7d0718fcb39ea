// The random-bit-flip decisions of the injector over one span of a tensor,
// by the threads of one 256-thread block (the RBF error model of Section
// II-B, used by Inject() in Algorithms 1 and 2; the same decisions drive the
// random-zero and random-NaN models at a rate).  Shared by the injection
// kernel and by the chunk pass that injects and signs in one sweep.
//
// Element i of a tensor flips iff its 64-bit uniform U_i is below
// T = floor(rate * 2^64) (every element when rate >= 1).  U_i is built from
// Philox4x32-10 (Salmon et al., SC'11) keyed by the seed, block c of stream s
// at counter (lo32(c), hi32(c), s, 0):
//   top byte    = byte (i mod 16) of block i/16 of stream 0
//   low 56 bits = 64-bit word (i mod 2) of block i/2 of stream 1
// A flipped element toggles the j-th lowest set bit of the mask with
// j = floor(y * popcount(mask) / 2^32), y = word 0 of block i of stream 2.
//
// For T < 2^56 an element can only flip when its top byte is 0, so each lane
// draws two blocks per 32 elements and evaluates the low bits only for the
// (1 in 256) elements whose top byte is zero.  Most groups of 32 (88 in 100)
// have none: a test of the whole group (two operations per word) queues the
// others, whose blocks are drawn again, 64 groups at a time, to find the
// elements.  VALU-bound; with the exact byte masks of every group instead the
// kernel took 96 us for 24 f32 [4096, 4096] tensors (four waves per compute unit
// then), now 55 us, 7.3 T elements/s.  The tensor is
// read and written only at flipped elements.
#pragma once

#include "philox.h"

namespace peat {
namespace {

// Per-wave queues: elements whose top byte is zero, then groups of 32 with
// such elements; each holds fewer than 64 left over and one append per lane.
constexpr int kQCand = 128, kQCap = 2 * kQCand;

// Random values (PEAT_MODEL_VALUE) listed by the injection kernel and written
// once it has ended, so that every source is read before any element changes.
struct InjList {
    uint2 *at;                   // (element within the segment, bits)
    uint32_t cap;
    uint32_t *n;                 // LDS counter
    uint64_t s0;                 // first element of the segment
};

// The chosen element's new bits: a bit flip, +0, the type's quiet NaN, a
// value of the tensor before the call (read from the copy d.src) or a
// uniformly random bit pattern.
// ATOMIC: the bit flip is one device-scope atomic XOR on the aligned 32-bit
// word that holds the element, performed in L2 (a 16-bit neighbour in the
// same word is XORed with zeros, so no other element can lose an update).
// The fused chunk pass reads the flipped lines right after its own flips;
// the host admits only batches whose test lines no other block reads, so no
// compute unit holds a copy of such a line from before the flip.
template <bool ATOMIC>
__device__ __forceinline__ void flip(const InjDesc &d, uint64_t i, const InjList &list) {
    if (d.model == PEAT_MODEL_BITFLIP) {
        const int b = chosen_bit(d.seed, d.mask, d.popc, i);
        if constexpr (ATOMIC) {
            const uintptr_t a = reinterpret_cast<uintptr_t>(d.x) + i * (d.dtype == PEAT_F32 ? 4 : 2);
            const uint32_t bit = (1u << b) << ((a & 2) * 8);
            __hip_atomic_fetch_xor(reinterpret_cast<uint32_t *>(a & ~uintptr_t(3)), bit, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        } else if (d.dtype == PEAT_F32) {
            uint32_t *p = static_cast<uint32_t *>(d.x) + i;
            *p ^= 1u << b;
        } else {
            uint16_t *p = static_cast<uint16_t *>(d.x) + i;
            *p = (uint16_t)(*p ^ (1u << b));
        }
    } else {
        uint32_t v;
        if (d.model == PEAT_MODEL_VALUE || d.model == PEAT_MODEL_UNIFORM) {
            // block i of stream 4: word 0 (64 bits) picks the source, word 2
            // is the uniform bit pattern
            uint32_t V[4];
            philox(i, 4, d.seed, V);
            if (d.model == PEAT_MODEL_VALUE) {
                const uint64_t s = __umul64hi(block_word64(V, 0), (uint64_t)d.n);
                const void *src = d.list_cap ? d.x : d.src;
                v = d.dtype == PEAT_F32 ? static_cast<const uint32_t *>(src)[s]
                                        : static_cast<const uint16_t *>(src)[s];
                if (d.list_cap) {
                    const uint32_t q = atomicAdd(list.n, 1u);
                    if (q < list.cap) {
                        list.at[q] = make_uint2((uint32_t)(i - list.s0), v);
                        return;
                    }
                    // (the capacity is 40 standard deviations above the mean)
                }
            } else {
                v = V[2];
            }
        } else {
            const bool nan = d.model == PEAT_MODEL_NAN;
            v = nan ? (d.dtype == PEAT_F32 ? 0x7FC00000u : (d.dtype == PEAT_F16 ? 0x7E00u : 0x7FC0u)) : 0u;
        }
        if (d.dtype == PEAT_F32)
            static_cast<uint32_t *>(d.x)[i] = v;
        else
            static_cast<uint16_t *>(d.x)[i] = (uint16_t)v;
    }
}

// Low 56 bits of U_i for a queued candidate (its top byte is 0, so U_i is
// just these bits): flip the element when they are below T.
template <bool ATOMIC>
__device__ __forceinline__ uint32_t settle_candidate(const InjDesc &d, uint64_t i, const InjList &list) {
    uint32_t B[4];
    philox(i >> 1, 1, d.seed, B);
    const uint64_t low = block_word64(B, (uint32_t)(i & 1)) & ((uint64_t(1) << 56) - 1);
    if (low < d.T) {
        flip<ATOMIC>(d, i, list);
        return 1;
    }
    return 0;
}

// The flips of elements [s0, s0 + len) of tensor d (s0 a multiple of 32, no
// multiple of 2^36 inside), made by the block's threads; queue holds the
// per-wave LDS queues.  Returns the calling thread's share of the flip count.
template <bool ATOMIC>
__device__ uint32_t inject_span(const InjDesc &d, uint64_t s0, uint64_t len, uint32_t (*queue)[kQCap],
                                const InjList &list) {
    const uint64_t n = (uint64_t)d.n;
    const uint32_t ngroups = (uint32_t)((len + 31) / 32);
    const uint64_t q0 = s0 >> 5;
    const uint64_t T = d.T;
    const int lane = threadIdx.x & 63;
    uint32_t flips = 0;

    if (!d.all && T < (uint64_t(1) << 56)) {
        uint32_t *cands = queue[threadIdx.x >> 6], *groups = cands + kQCand;   // span-relative elements, groups
        uint32_t qn = 0, gn = 0;                           // wave-uniform
        const uint32_t clo = (uint32_t)(2 * q0), chi = __builtin_amdgcn_readfirstlane((uint32_t)((2 * q0) >> 32));
        auto below = [&](uint64_t m) {                     // lanes of m before this one
            return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        };
        auto settle = [&](uint32_t cnt) {                  // the last cnt candidates, one per lane
            qn -= cnt;
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            if ((uint32_t)lane < cnt) flips += settle_candidate<ATOMIC>(d, s0 + cands[qn + lane], list);
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        };
        auto expand = [&](uint32_t cnt) {                  // the elements of the last cnt groups
            gn -= cnt;
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            uint32_t cand = 0, g = 0;
            if ((uint32_t)lane < cnt) {
                g = groups[gn + lane];
                // the 32 top bytes of the group: blocks 2(q0+g) and 2(q0+g)+1
                uint32_t A[8];
                philox0(clo + 2 * g, chi, d.seed, A);
                philox0(clo + 2 * g + 1, chi, d.seed, A + 4);
                // exact zero-byte mask of each word: bit 7 of a byte is set
                // iff the byte is zero; one multiply gathers bits 7, 15, 23,
                // 31 into bits 28..31 (the other partial products land on
                // distinct lower bits, so nothing carries)
#pragma unroll
                for (int w = 0; w < 8; ++w) {
                    const uint32_t v = A[w];
                    const uint32_t z = ~(((v & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | v | 0x7F7F7F7Fu);
                    cand |= ((z * 0x00204081u) >> 28) << (4 * w);
                }
                const uint64_t rest = len - ((uint64_t)g << 5);
                if (rest < 32) cand &= (1u << (uint32_t)rest) - 1u;   // ragged end
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
            // one element per lane and round
            while (true) {
                const uint64_t m = __ballot(cand != 0);
                if (m == 0) break;
                if (cand != 0) {
                    cands[qn + below(m)] = (g << 5) | (uint32_t)(__ffs(cand) - 1);
                    cand &= cand - 1;
                }
                qn += (uint32_t)__popcll(m);
                if (qn >= 64) settle(64);
            }
        };
        const uint32_t iters = (ngroups + kBlock - 1) / kBlock;
        for (uint32_t k = 0; k < iters; ++k) {
            const uint32_t g = k * kBlock + threadIdx.x;
            uint32_t A[8], some = 0;
            philox0(clo + 2 * g, chi, d.seed, A);
            philox0(clo + 2 * g + 1, chi, d.seed, A + 4);
            // a byte borrows from bit 7 of (v - 1 per byte) & ~v exactly if some byte is zero
#pragma unroll
            for (int w = 0; w < 8; ++w) some |= (A[w] - 0x01010101u) & ~A[w];
            const bool has = (some & 0x80808080u) != 0 && g < ngroups;
            const uint64_t m = __ballot(has);
            if (has) groups[gn + below(m)] = g;
            gn += (uint32_t)__popcll(m);
            if (gn >= 64) expand(64);
        }
        if (gn != 0) expand(gn);
        if (qn != 0) settle(qn);
    } else {
        // general threshold (rate >= 2^-8) or every element
        const uint64_t Ttop = T >> 56, Tlow = T & ((uint64_t(1) << 56) - 1);
        for (uint32_t g = threadIdx.x; g < ngroups; g += kBlock) {
            const uint64_t q = q0 + g;
            uint32_t A[8];
            if (!d.all) {
                philox(2 * q, 0, d.seed, A);
                philox(2 * q + 1, 0, d.seed, A + 4);
            }
            const uint64_t ibase = q << 5;
            const uint64_t end = s0 + len < n ? s0 + len : n;
            const uint32_t cnt = (end - ibase) < 32 ? (uint32_t)(end - ibase) : 32u;
            for (uint32_t b = 0; b < cnt; ++b) {
                const uint64_t i = ibase + b;
                bool f = d.all;
                if (!f) {
                    const uint64_t top = (A[b >> 2] >> (8 * (b & 3))) & 0xFF;
                    if (top < Ttop) {
                        f = true;
                    } else if (top == Ttop) {
                        uint32_t B[4];
                        philox(i >> 1, 1, d.seed, B);
                        f = (block_word64(B, (uint32_t)(i & 1)) & ((uint64_t(1) << 56) - 1)) < Tlow;
                    }
                }
                if (f) {
                    flip<ATOMIC>(d, i, list);
                    ++flips;
                }
            }
        }
    }
    return flips;
}

}  // namespace
}  // namespace peat
