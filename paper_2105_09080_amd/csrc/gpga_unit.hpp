// Column units: the 4, 2 or 1 consecutive columns one lane owns in every row, and how lanes map to them.
//
// Rows need no more than the 4-byte alignment of a float: gfx950 takes 16-byte global accesses at any 4-byte
// aligned address, so leading dimensions and bases that no vector width divides run on the same wide lanes as
// aligned ones (only the 128-byte lines a wavefront touches go from 8 to 9 per row segment).
//
// When the column count is no multiple of the lane width, the last unit is moved left until it ends at the last
// column.  It then overlaps the unit before it: both lanes compute the shared columns from the same values and
// store the same bits.  m is updated in place, so the two lanes must be in one wavefront, where they read a row
// in one instruction and store it in a later one; should the last unit open a tile of its own, all units are
// shifted one lane to the right (`lead`) and lane 0 of the first tile doubles unit 0 in the same way.
#pragma once

#include "gpga_internal.hpp"

typedef float v4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float v2u __attribute__((ext_vector_type(2), aligned(4)));

template <typename T>
struct Unit;
template <>
struct Unit<v4f> {
    typedef v4u mem;
};
template <>
struct Unit<v2f> {
    typedef v2u mem;
};
template <>
struct Unit<float> {
    typedef float mem;
};

// Streaming (non-temporal) access to the unit at p.
template <typename T>
__device__ __forceinline__ T ld_unit(const float* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const typename Unit<T>::mem*>(p));
}
template <typename T>
__device__ __forceinline__ void st_unit(float* p, const T& v) {
    __builtin_nontemporal_store(v, reinterpret_cast<typename Unit<T>::mem*>(p));
}
// Cached read.
template <typename T>
__device__ __forceinline__ T ld_unit_cached(const float* p) {
    return *reinterpret_cast<const typename Unit<T>::mem*>(p);
}

// First column of the unit that lane `lane` of a tile of `width` lanes owns (T = v4f, v2f or float).
template <typename T>
__device__ __forceinline__ int64_t unit_column(const StepGeom& ge, int64_t tile, int width, int lane) {
    constexpr int V = sizeof(T) / sizeof(float);
    int64_t c = (tile * width + lane - ge.lead) * V;
    if (c < 0) c = 0;
    return c > ge.d - V ? ge.d - V : c;
}
__device__ __forceinline__ bool unit_on(const StepGeom& ge, int64_t tile, int width, int lane) {
    return tile * width + lane - ge.lead < ge.ncols;
}
// Whether every lane of the tile owns a unit.
__device__ __forceinline__ bool whole_units(const StepGeom& ge, int64_t tile, int width) {
    return (tile + 1) * width - ge.lead <= ge.ncols;
}
// Host side: the units of d columns for lanes of V columns in tiles of `width` lanes.
inline void set_units(StepGeom* ge, int V, int width) {
    ge->ncols = (ge->d + V - 1) / V;
    ge->lead = (ge->d % V != 0 && ge->ncols % width == 1) ? 1 : 0;
}
inline int64_t unit_tiles(const StepGeom& ge, int width) { return (ge.ncols + ge.lead + width - 1) / width; }
