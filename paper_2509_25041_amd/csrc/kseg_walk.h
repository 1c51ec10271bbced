// Weight offsets of a lane that walks a K axis cut in segments (shared experts' down projection), for buffer loads.
// Plain C++ (constexpr: host and device), so that the arithmetic can be checked on the host.
#pragma once
#include <cstdint>

namespace grace {

constexpr uint32_t NO_DATA = 0x80000000u;   // an offset past the range of the buffer descriptors: reads nothing, gives zeros

// The lane looks at positions k, k + step, ... of K; what the segments before a position add to its byte offset
// beyond el * k is `jump` (elements of el bytes).
struct KSegWalk {
    int pos;            // position in the K segment
    uint32_t jump = 0;

    // bytes to add to the offset of position k, then one step on.  Past K there is no data, whatever `jump` has grown to
    // (in 32 bits it wraps there when the weights hold 2 GiB or more).
    constexpr uint32_t next(int k, int K, int seg_len, int64_t seg_stride, int step, int el = 2) {
        while (pos >= seg_len) {
            pos -= seg_len;
            jump += (uint32_t)((seg_stride - seg_len) * el);
        }
        pos += step;
        return k < K ? jump : NO_DATA;
    }
};

// k / len for k below 2^31 by one multiplication, for lanes that keep nothing from step to step: with 2^(31+b) = q len + r, b the bits
// that len - 1 takes, the factor q + 1 is too large by less than len / len, which moves no quotient (k (len - r) < 2^(31+b)).
struct KSegDiv {
    uint32_t factor;
    int shift;
    constexpr explicit KSegDiv(int len) : factor(0), shift(0) {   // len >= 2
        int b = 1;
        while ((uint32_t)len > (uint32_t)1 << b) ++b;
        factor = (uint32_t)(((uint64_t)1 << (31 + b)) / (uint32_t)len + 1);
        shift = b - 1;
    }
    constexpr uint32_t operator()(int k) const { return (uint32_t)(((uint64_t)(uint32_t)k * factor) >> 32) >> shift; }
};

// offset + add, or no data where either has none
constexpr uint32_t offset_with(uint32_t offset, uint32_t add) { return (offset + add) | (offset & NO_DATA) | (add & NO_DATA); }

}  // namespace grace
