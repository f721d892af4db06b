/*
 * qm_stream.hpp -- how the kernels that read an array walk it: wave tiles of
 * 16-byte vectors (streaming and batch kernels; the generating ones, which
 * have no input, share the vector types and the launch rules).
 */
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "qm_internal.h"

namespace qm {

typedef double d2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T> struct vec16;
template <> struct vec16<double> { typedef d2 type; static constexpr int n = 2; };
template <> struct vec16<float> { typedef f4 type; static constexpr int n = 4; };

/* The same 16 bytes at the alignment of an element: gfx950 takes a dwordx4
   access at any dword. */
template <typename T> struct vec16any;
template <> struct vec16any<double> { typedef double type __attribute__((ext_vector_type(2), aligned(8))); };
template <> struct vec16any<float> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };

/* The first lane's value of x, as a wave-uniform (scalar) value. */
__device__ __forceinline__ uint64_t wave_uniform(uint64_t x)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint32_t wave_lane()
{
    return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
}

/*
 * An array pair cut into a body of nvec 16-byte vectors and fewer than two
 * vectors' worth of edge elements, [0, head) and [tail, n).  The body starts
 * on a 16-byte boundary of the output; the input may lie at any element (its
 * 16-byte loads then straddle boundaries, which costs a little of the load
 * rate, where reading element by element would cost half of it).
 */
template <typename T>
struct Span {
    const T* in;
    T* out;
    uint64_t head, nvec, tail, n;
};

template <typename T>
__host__ __device__ __forceinline__ Span<T> make_span(const T* in, T* out, uint64_t n)
{
    constexpr int NV = 16 / sizeof(T);
    Span<T> s;
    s.in = in;
    s.out = out;
    s.n = n;
    s.head = ((16 - (reinterpret_cast<uintptr_t>(out) % 16)) % 16) / sizeof(T);
    if (s.head > n) s.head = n;
    s.nvec = (n - s.head) / NV;
    s.tail = s.head + s.nvec * NV;
    return s;
}

/*
 * One wave's walk over a span: tiles of 64 UNROLL consecutive vectors (lane
 * l reads vector l of each 1 KB row), dealt out to nwaves waves in turn,
 * non-temporal both ways (each byte is touched once).  Measured on MI355X
 * these wave-contiguous tiles stream 2-10% faster than a grid-stride layout.
 * Only the span's last tile can be partial, and whole waves enter it
 * together (the maps' wave votes need every lane).  begin() issues the first
 * tile's loads, so that they are in flight while a kernel stages its table.
 *
 * Map: tile(const T (&x)[K], T (&y)[K]) for the K elements a lane holds, and
 * one(T) for an edge element.
 */
template <typename T, int UNROLL>
struct Walk {
    typedef typename vec16<T>::type V;
    typedef typename vec16any<T>::type VA;
    static constexpr int NV = vec16<T>::n;
    static constexpr int K = NV * UNROLL;
    static constexpr uint64_t TILE = 64ull * UNROLL;

    V x[UNROLL];
    uint64_t t, step;

    __device__ __forceinline__ void load(const Span<T>& s, uint32_t lane)
    {
        const VA* vin = reinterpret_cast<const VA*>(s.in + s.head);
        if (t + TILE <= s.nvec) {
#pragma unroll
            for (int k = 0; k < UNROLL; ++k) x[k] = __builtin_nontemporal_load(vin + t + 64 * k + lane);
        }
    }

    __device__ __forceinline__ void begin(const Span<T>& s, uint64_t wave, uint64_t nwaves, uint32_t lane)
    {
        t = wave * TILE;
        step = nwaves * TILE;
        load(s, lane);
    }

    template <class Map>
    __device__ __forceinline__ void eval(const V (&v)[UNROLL], V (&y)[UNROLL], const Map& map)
    {
        T u[K], w[K];
#pragma unroll
        for (int k = 0; k < UNROLL; ++k)
#pragma unroll
            for (int j = 0; j < NV; ++j) u[NV * k + j] = v[k][j];
        map.tile(u, w);
#pragma unroll
        for (int k = 0; k < UNROLL; ++k)
#pragma unroll
            for (int j = 0; j < NV; ++j) y[k][j] = w[NV * k + j];
    }

    template <class Map>
    __device__ __forceinline__ void run(const Span<T>& s, uint32_t lane, const Map& map)
    {
        const VA* vin = reinterpret_cast<const VA*>(s.in + s.head);
        V* vout = reinterpret_cast<V*>(s.out + s.head);
        while (t + TILE <= s.nvec) {
            V y[UNROLL];
            eval(x, y, map);
#pragma unroll
            for (int k = 0; k < UNROLL; ++k) __builtin_nontemporal_store(y[k], vout + t + 64 * k + lane);
            t += step;
            load(s, lane);
        }
        if (t < s.nvec) {
            V y[UNROLL];
#pragma unroll
            for (int k = 0; k < UNROLL; ++k) {
                const uint64_t i = t + 64 * k + lane;
                x[k] = (V)(T)0.5;
                if (i < s.nvec) x[k] = __builtin_nontemporal_load(vin + i);
            }
            eval(x, y, map);
#pragma unroll
            for (int k = 0; k < UNROLL; ++k) {
                const uint64_t i = t + 64 * k + lane;
                if (i < s.nvec) __builtin_nontemporal_store(y[k], vout + i);
            }
        }
    }
};

/* The edge elements of a span, by one workgroup. */
template <typename T, class Map>
__device__ __forceinline__ void run_edges(const Span<T>& s, const Map& map)
{
    const uint64_t extra = s.head + (s.n - s.tail);
    for (uint64_t e = threadIdx.x; e < extra; e += blockDim.x) {
        const uint64_t i = e < s.head ? e : s.tail + (e - s.head);
        s.out[i] = map.one(s.in[i]);
    }
}

/*
 * A large launch over a table of more than 24 KB in LDS: a workgroup for every
 * tile or two would stage more than the 16 KB that it reads, so such a launch
 * keeps a grid of a few workgroups per unit, with four vectors per lane.
 * MI355X, us, two tiles each -> fixed grid: FP64 hyperbolic (1, 0, 1e-6), 41
 * KB, 2^27 517 -> 374 at 16 per unit, (1, 0.9, 5), 27 KB, 412 -> 380; FP64
 * Student t nu = 0.3, 51 KB, 713 -> 523 at 2 per unit, nu = 0.4, 29 KB, 2^25 99
 * -> 92, 2^27 387 -> 388; FP32 nu = 0.3, 32 KB, 207 -> 185.
 */
constexpr int T_TABLE_BLOCKS = 2, H_TABLE_BLOCKS = 16;
inline void fit_to_table(KernelShape& ks, size_t lds_bytes, int blocks_per_cu, int cus)
{
    if (lds_bytes <= 24 * 1024) return;
    ks.big_unroll = 4;
    ks.big_blocks = (uint64_t)blocks_per_cu * cus;
    ks.huge_vecs = 0;
}

/* launches of the last two kinds of KernelShape */
inline bool launch_big(uint64_t nvec, const KernelShape& ks) { return ks.big_vecs && nvec >= ks.big_vecs; }
inline bool launch_huge(uint64_t nvec, const KernelShape& ks) { return ks.huge_vecs && nvec >= ks.huge_vecs; }

/*
 * Vectors per lane for a launch of nvec vectors: the family's own, halved
 * while the grid would have fewer than two workgroups of 256 for each
 * compute unit; a big launch's own.  A short launch is bound by the latency of
 * one tile, which grows with the elements a lane holds, and by the compute
 * units left idle: on MI355X 2^17 FP64 hyperbolic samples took 4.3 us with
 * four vectors per lane and 3.3 with one, fused FP32 ones 7.5 and 3.7; at 2^20
 * (two workgroups per unit with four vectors) the three are within 5%.
 */
inline int launch_unroll(uint64_t nvec, const KernelShape& ks, int cus)
{
    if (ks.fixed_unroll) return ks.unroll;
    if (launch_huge(nvec, ks)) return 4;
    if (launch_big(nvec, ks)) return ks.big_unroll;
    int u = ks.unroll;
    while (u > 1 && nvec < 512ull * u * (uint64_t)cus) u /= 2;
    return u;
}

/*
 * Workgroups of a launch.  Few of them keep each one's set-up (a staged
 * table) small against its work, and for arrays that the last-level cache
 * holds that is best (FP64 hyperbolic samples, 2^24: 46 us with 3 workgroups
 * per compute unit, 55 with 64).  Large arrays run at the memory's rate, and
 * there a workgroup takes two tiles, one from each half of the array: the
 * resident workgroups, handed out in order, then write two windows that
 * advance together, where a fixed grid's strides spread them over the array
 * more and more, and the second tile's loads are in flight while the first is
 * mapped.  MI355X, us, fixed grid -> two tiles: FP64 quantiles 2^28 752 ->
 * 705, 2^29 1620 -> 1430 (both faster than a copy kernel on a fixed grid:
 * 732 for 2^28); FP64 Student t 2^26 174.5 -> 167.5, 2^27 354 -> 340; FP64
 * hyperbolic 2^27 363 -> 346; FP32 Student t 2^28 362 -> 340.  One tile each
 * is slower there (Student t 2^26 187, quantiles 182 against 172), and two
 * neighbouring tiles are too at some sizes (quantiles 2^28 741).  Each family
 * changes over where the two tiles have overtaken its fixed grid, at 256 MB to
 * 1 GB of one array.  From 2 GB on one tile of four vectors each does better
 * for some (us, two tiles -> one; FP64 2^28): quantiles 771 -> 755 on the
 * mixture and 751 -> 683 on uniforms, exp -> normal 688 -> 677, Student t nu =
 * 30 742 -> 705 and nu = 4 706 -> 708; FP32 2^29: Student t 718 -> 690 (nu = 1
 * 725 -> 726), hyperbolic 729 -> 715, variance-gamma 740 -> 727.  It costs
 * where more is staged for the one tile (FP64 hyperbolic 703 -> 739, Student t
 * with rows of 16, nu = 1, 706 -> 771) and gives nothing to the FP32 quantiles
 * (783 -> 794, 724 -> 724) and exp -> normal (821 -> 822): those keep two.
 */
inline unsigned launch_blocks(uint64_t nvec, int unroll, const KernelShape& ks)
{
    const uint64_t per_block = 256ull * unroll, tiles = (nvec + per_block - 1) / per_block;
    const bool big = launch_big(nvec, ks);
    const uint64_t blocks = big && !launch_huge(nvec, ks) ? (tiles + 1) / 2 : tiles;
    const uint64_t cap = big ? ks.big_blocks : ks.max_blocks;
    return (unsigned)(blocks > cap ? cap : blocks < 1 ? 1 : blocks);
}

/* f(std::integral_constant<int, u>) for u = 1, 2 or 4. */
template <class F>
inline void with_unroll(int u, F f)
{
    if (u == 4) f(std::integral_constant<int, 4>());
    else if (u == 2) f(std::integral_constant<int, 2>());
    else f(std::integral_constant<int, 1>());
}

}  // namespace qm
