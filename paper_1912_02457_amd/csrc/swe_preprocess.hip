// Preprocessing of the input fields on the device, before a domain is
// created: bathymetry at the cell intersections from cell values (section
// "Bathymetry"), erosion of the land mask (same section), and factor-two
// refinement and coarsening of cell fields, land mask and corner depths
// (section "Refinement and coarsening of grid").  Device pointers in and out,
// asynchronous on the caller's stream, no device memory of the library's own.
// Beside them, the kernel that copies a domain's state planes out.
#include <cmath>
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <mutex>
#include <string>

#include "swe_host.h"

namespace {

using swe::set_error;

// ---------------------------------------------------------------------------
// Bathymetry reconstruction, one launch per round.
//   round 0 (INIT): corners = the average over the water cells meeting there
//     of each cell's limited plane evaluated at the corner (eqs. recon_1-3)
//     applied to the cell values themselves;
//   round k >= 1: misfit dH = Hm - (mean of the cell's corners) on water
//     cells, its corner estimate by the same three equations added to the
//     corners, then H <- (1 - w) H + (w/4) (sum of the 4 neighbours) with a
//     neighbour outside the domain replaced by the corner itself.
// Corners that touch no water cell hold the mean of the four cell values
// around them (edge cells repeated).
//
// Work decomposition: one wave per (strip, row segment).  Lane l holds
// corner column I = 58 s - 3 + l and cell column i = I (the cell to the
// upper right of the corner); an output corner reads columns I-3 .. I+3, so
// lanes 3..60 store and the six others are halo.  The wave walks up the
// rows with a register pipeline: the step that loads corner row a and cell
// row a-1 computes the misfit of cell row a-1, the slopes and corner
// contributions of cell row a-2, the corrected corners of row a-2 and the
// smoothed output row a-3.  Neighbouring columns come through DPP lane
// shifts.  Two rounds to a launch double the halo (strips of 52, lanes 6..57)
// and the warm-up rows and halve the launches and the corners' traffic.
//
// What bounds a round is the launch on small grids and memory (13 bytes a
// corner) on large ones, once the instructions of a row are few: water flags
// are 64-bit scalars of a row, shifted and counted on the scalar unit, the
// limiter is one median, addresses are buffer accesses with a scalar row
// offset, and a segment with no row or lane outside the domain has a body
// without the tests for it.  29 vector instructions a row and round, 71
// before; microseconds a round with the rounds one by one before that, one by
// one after it, and in pairs: 100 x 100 5.5, 4.1 and 2.8; 1202 x 602 6.8, 5.5
// and 4.4; 2600 x 900 11.1, 7.9 and 7.5; 4000 x 2400 31.7, 20.6 (6.1 TB/s)
// and 17.4.
constexpr int halo(bool pair) { return pair ? 6 : 3; }  // columns and rows on each side
constexpr int strip(bool pair) { return 64 - 2 * halo(pair); }

constexpr int kDppShl1 = 0x130;  // wave_shl:1 -- value of lane + 1
constexpr int kDppShr1 = 0x138;  // wave_shr:1 -- value of lane - 1
// 0 past the ends of the wave; in this form the shift joins the instruction
// that uses it
__device__ __forceinline__ float lane_right(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kDppShl1, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_left(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kDppShr1, 0xF, 0xF, true));
}

using Mask = uint64_t;  // bit l = lane l
__device__ __forceinline__ bool in(Mask m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Element access through a 32-bit byte offset from a uniform base pointer
// (the scalar-base + vector-offset addressing form; no 64-bit address
// arithmetic per lane).  Every plane stays below 4 GiB.
__device__ __forceinline__ float ldf(const float *__restrict__ base, uint32_t i)
{
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(base) + (i << 2));
}
__device__ __forceinline__ int ldb(const uint8_t *__restrict__ base, uint32_t i)
{
    return *reinterpret_cast<const uint8_t *>(reinterpret_cast<const char *>(base) + i);
}
__device__ __forceinline__ void stf(float *__restrict__ base, uint32_t i, float v)
{
    *reinterpret_cast<float *>(reinterpret_cast<char *>(base) + (i << 2)) = v;
}

// The limited slope of two differences: the smaller one where both have one
// sign, else 0, which is the median of the two and 0.  The median of a NaN is
// not 0: a difference is taken through `difference`, which makes it 0.
__device__ __forceinline__ float minmod2(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0.0f); }
__device__ __forceinline__ float difference(Mask both, float a, float b)
{
    const float d = a - b;
    return in(both & __builtin_amdgcn_ballot_w64(d == d)) ? d : 0.0f;
}

// Blocks go to the 8 XCDs round-robin; give each XCD a contiguous run of
// blocks so that neighbouring strips and segments share lines in one L2.
__device__ __forceinline__ int xcd_block(int b, int n)
{
    int q = n >> 3, r = n & 7, x = b & 7, k = b >> 3;
    return x * q + min(x, r) + k;
}

// this wave's work item, the same in all its lanes
__device__ __forceinline__ int wave_item()
{
    return xcd_block(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y) * 4 +
           __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// A plane as a buffer: an access adds a scalar row offset and a lane's column
// offset in the load itself, so an address costs no vector instruction.
// Every plane stays below 4 GiB; accesses past its end read 0 or are dropped.
struct Plane {
    __amdgpu_buffer_rsrc_t r;
    uint32_t pitch;  // bytes of a row
    __device__ __forceinline__ Plane(const void *p, uint32_t row_bytes, uint32_t rows)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)(row_bytes * rows), 0x00020000)),
          pitch(row_bytes)
    {
    }
    __device__ __forceinline__ float f32(int row, uint32_t col) const
    {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, col << 2, (uint32_t)row * pitch, 0));
    }
    __device__ __forceinline__ int byte(int row, uint32_t col) const
    {
        return (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(r, col, (uint32_t)row * pitch, 0);
    }
    __device__ __forceinline__ void put(int row, uint32_t col, float v) const
    {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, col << 2, (uint32_t)row * pitch, 0);
    }
};

// Lanes of a wave at or beyond the first and last corner column.
struct SideLanes { Mask west, east; };

// One round of a wave as a pipeline over its rows: `next` takes corner row a
// and cell row a-1 (values, water flags) and gives row a-3 of the round's
// result, from the seventh row on.  INSIDE: no lane or row lies outside the
// domain.  Names give the row relative to the newest corner row a.
template <bool INIT, bool INSIDE>
struct Round {
    float H1 = 0.f, H2 = 0.f, S1 = 0.f;   // corners a-1, a-2; sum of corner a-1 and its right neighbour
    float D2 = 0.f, Y2 = 0.f;             // misfit of cell row a-2 (0 off the water); its difference to row a-3
    Mask W2 = 0;                          // water flags of cell row a-2
    Mask X3 = 0, B3 = 0, O3 = 0, O4 = 0;  // rows a-3, a-4: one, both, any of a cell and its left neighbour water
    float UR3 = 0.f, UL3 = 0.f;           // cell row a-3: estimates at its upper corners
    float P3 = 0.f, P4 = 0.f;             // corrected corners of rows a-3, a-4
    float M1 = 0.f, N2 = 0.f, N3 = 0.f;   // cell values, row a-2; sum with the left neighbour, rows a-3, a-4

    __device__ __forceinline__ float next(int a, int ny, const SideLanes &side, float w, float Ha, float Mc, Mask W1)
    {
        // misfit of cell row a-1
        const float S0 = lane_right(Ha) + Ha;
        const float misfit = INIT ? Mc : __builtin_fmaf(-0.25f, S1 + S0, Mc);
        const float D1 = in(W1) ? misfit : 0.f;

        // slopes and corner estimates of cell row a-2; all 0 off the water
        const float Dr = lane_right(D2);
        const float dx = difference(W2 & (W2 >> 1), Dr, D2), Y1 = difference(W2 & W1, D1, D2);
        const float sx = 0.5f * minmod2(lane_left(dx), dx), sy = 0.5f * minmod2(Y2, Y1);
        const float U = D2 + sy, L = D2 - sy;
        const float UR2 = U + sx, UL2 = U - sx, DR2 = L + sx, DL2 = L - sx;

        // corrected corner row a-2: the mean over the water cells among
        // (a-3, I-1), (a-3, I), (a-2, I-1), (a-2, I).  Cells off the water add
        // 0; the number of water cells is summed bit by bit in the masks
        const Mask W2l = W2 << 1, X2 = W2 ^ W2l, B2 = W2 & W2l, O2 = W2 | W2l;
        const Mask odd = X3 ^ X2, two = B3 ^ B2 ^ (X3 & X2), four = B3 & B2;
        const float acc = lane_left(UR3) + UL3 + (lane_left(DR2) + DL2);
        float share = in(four) ? 0.25f : 1.0f;
        share = in(two) ? 0.5f : share;
        share = in(two & odd) ? 1.0f / 3.0f : share;
        const float P2 = INIT ? acc * share : __builtin_fmaf(acc, share, H2);

        // result row Y = a-3
        const int Y = a - 3;
        const float N1 = lane_left(M1) + M1;
        float out = P3;
        if (!INIT) {
            const float up = (INSIDE || Y < ny) ? P2 : P3, down = (INSIDE || Y > 0) ? P4 : P3;
            float left = lane_left(P3), right = lane_right(P3);
            if (!INSIDE) {
                left = in(side.west) ? P3 : left;
                right = in(side.east) ? P3 : right;
            }
            out = __builtin_fmaf(1.0f - w, P3, 0.25f * w * ((up + down) + left + right));
        }
        float fill = 0.25f * (N3 + N2);
        asm("" : "+v"(out), "+v"(fill));  // both computed, then chosen: no branch
        out = in(O4 | O3) ? out : fill;

        H2 = H1; H1 = Ha; S1 = S0;
        D2 = D1; Y2 = Y1;
        W2 = W1; X3 = X2; B3 = B2; O4 = O3; O3 = O2;
        UR3 = UR2; UL3 = UL2;
        P4 = P3; P3 = P2;
        N3 = N2; N2 = N1; M1 = Mc;
        return out;
    }
};

// A segment of R rows through one round or, with PAIR, through two: the second
// takes the rows of the first three steps later, so the corners between the
// two never leave the wave.
template <bool INIT, bool PAIR, bool INSIDE, int R>
__device__ __forceinline__ void recon_rows(int nx, int ny, int J0, int I0, const float *__restrict__ Hm,
                                           const uint8_t *__restrict__ land, const float *__restrict__ Hin, float w,
                                           float *__restrict__ Hout)
{
    constexpr int H = halo(PAIR), NS = R + 2 * H;  // steps: H warm-up rows below, H above
    const int lane = threadIdx.x & 63, I = I0 + lane;
    const uint32_t Ic = (uint32_t)(INSIDE ? I : min(max(I, 0), nx));
    const uint32_t ic = (uint32_t)(INSIDE ? I : min(max(I, 0), nx - 1));
    const uint32_t nxc = (uint32_t)nx + 1;
    const Plane corners_in(Hin, nxc * 4u, (uint32_t)ny + 1), corners_out(Hout, nxc * 4u, (uint32_t)ny + 1);
    const Plane cells(Hm, (uint32_t)nx * 4u, (uint32_t)ny), mask(land, (uint32_t)nx, (uint32_t)ny);
    const Mask cols = INSIDE ? ~(Mask)0 : __builtin_amdgcn_ballot_w64(I >= 0 && I < nx);
    const SideLanes side{__builtin_amdgcn_ballot_w64(I <= 0), __builtin_amdgcn_ballot_w64(I >= nx)};
    const int a0 = J0 - H;

    // every load of the segment first (clamped rows: always valid
    // addresses), so the wave waits for memory once, not once per row; a row's
    // base is scalar, a lane adds its column
    float Hb[NS], Mb[NS];
    int Lb[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        const int rc = INSIDE ? a0 + k : min(max(a0 + k, 0), ny);
        const int rm = INSIDE ? a0 + k - 1 : min(max(a0 + k - 1, 0), ny - 1);
        Hb[k] = INIT ? 0.f : corners_in.f32(rc, Ic);
        Mb[k] = cells.f32(rm, ic);
        Lb[k] = 0;
    }
    if (land) {
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            const int rm = INSIDE ? a0 + k - 1 : min(max(a0 + k - 1, 0), ny - 1);
            Lb[k] = mask.byte(rm, ic);
        }
    }
    // all of them have arrived here: without this the compiler moves a row's
    // loads to where the row is used, one wait each
#pragma unroll
    for (int k = 0; k < NS; ++k) asm volatile("" : "+v"(Hb[k]), "+v"(Mb[k]), "+v"(Lb[k]));

    const auto water = [&](int k) -> Mask {
        const int j = a0 + k - 1;
        return (INSIDE || (j >= 0 && j < ny)) ? cols & __builtin_amdgcn_ballot_w64(Lb[k] == 0) : 0;
    };
    Round<INIT, INSIDE> first;
    Round<false, INSIDE> second;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        float out = first.next(a0 + k, ny, side, w, Hb[k], Mb[k], water(k));
        if (PAIR && k >= 6) out = second.next(a0 + k - 3, ny, side, w, out, Mb[k - 3], water(k - 3));
        const int Y = a0 + k - H;
        if (k >= 2 * H && lane >= H && lane < H + strip(PAIR) && (INSIDE || (I <= nx && Y <= ny)))
            corners_out.put(Y, (uint32_t)I, out);
    }
}

template <bool INIT, bool PAIR, int R>
__global__ __launch_bounds__(256) void recon_round_kernel(int nx, int ny, int nsx, int nitems,
                                                          const float *__restrict__ Hm,
                                                          const uint8_t *__restrict__ land,
                                                          const float *__restrict__ Hin, float w,
                                                          float *__restrict__ Hout)
{
    constexpr int H = halo(PAIR);
    const int item = wave_item();
    if (item >= nitems) return;  // whole waves leave together
    const int seg = item / nsx, J0 = seg * R, I0 = (item - seg * nsx) * strip(PAIR) - H;
    if (I0 >= 0 && I0 + 63 < nx && J0 > H && J0 + R + H - 2 < ny)
        recon_rows<INIT, PAIR, true, R>(nx, ny, J0, I0, Hm, land, Hin, w, Hout);
    else
        recon_rows<INIT, PAIR, false, R>(nx, ny, J0, I0, Hm, land, Hin, w, Hout);
}

int64_t div_up(int64_t a, int64_t b) { return (a + b - 1) / b; }

// four items to a block; a second grid dimension where the threads of one
// would leave 32 bits
dim3 item_grid(int64_t items)
{
    const int64_t blocks = div_up(items, 4), x = std::min<int64_t>(blocks, 1 << 20);
    return dim3((unsigned)x, (unsigned)div_up(blocks, x));
}

template <bool INIT, bool PAIR>
hipError_t launch_recon(hipStream_t s, int nx, int ny, const float *Hm, const uint8_t *land, const float *Hin, float w,
                        float *Hout)
{
    const int nsx = (nx + 1 + strip(PAIR) - 1) / strip(PAIR);
    // rows per segment, by the waves that 8 would give: 4 below 1.5 a SIMD (a
    // wave's rows are a serial chain), 16 from 12 a SIMD (fewer warm-up rows).
    // Microseconds a round of a pair with 4, 8 and 16 rows: 250 x 130 2.8, 3.5
    // and 5.0; 1202 x 602 4.6, 4.4 and 5.1; 2600 x 900 8.9, 7.5 and 7.9; 4000
    // x 2400 25.6, 18.5 and 17.4.  A round alone is never faster with 16 than 8.
    const int64_t waves = nsx * div_up((int64_t)ny + 1, 8);
    const int R = waves < 1536 ? 4 : PAIR && waves >= 12288 ? 16 : 8;
    const int64_t items = (int64_t)nsx * ((ny + 1 + R - 1) / R);
    auto *kernel = R == 4 ? recon_round_kernel<INIT, PAIR, 4> : R == 8 ? recon_round_kernel<INIT, PAIR, 8>
                 : recon_round_kernel<INIT, PAIR, PAIR ? 16 : 8>;
    hipLaunchKernelGGL(kernel, item_grid(items), dim3(256), 0, s, nx, ny, nsx, (int)items, Hm, land, Hin, w, Hout);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Erosion, refinement and coarsening: every byte is touched once, so memory
// is the bound and the kernels only have to keep enough of it in flight.  A
// wave takes a strip of columns and kRegridRows rows, issues all its loads
// before it uses the first, has the neighbours along x by lane shifts and
// those along y in registers, and holds the water flags of a row as one
// 64-bit scalar.  (Before, a thread loaded a cell's flags, waited, then loaded
// the neighbours those flags asked for, one cell at a time.)  2600 x 900 with
// three fields, microseconds before and now: erosion 24 and 13 to 18 (by what
// the caches hold), refinement 77 and 33, coarsening 14 and 9.4 (6.0, 6.0 and
// 4.8 TB/s).  Cells and corners of one call
// share a launch.  2 or 8 rows to a wave give the same.
//
// A vector access of several elements states the alignment of one element:
// rows of odd length and planes inside larger arrays are not aligned to more.
constexpr int kRegridRows = 4;

typedef float f32x2 __attribute__((ext_vector_type(2), aligned(4)));
typedef uint16_t u8x2 __attribute__((aligned(1)));

__device__ __forceinline__ f32x2 ldf2(const float *base, uint32_t i)
{
    return *reinterpret_cast<const f32x2 *>(reinterpret_cast<const char *>(base) + (i << 2));
}
__device__ __forceinline__ void stf2(float *base, uint32_t i, float x, float y)
{
    f32x2 v;
    v.x = x;
    v.y = y;
    *reinterpret_cast<f32x2 *>(reinterpret_cast<char *>(base) + (i << 2)) = v;
}
__device__ __forceinline__ uint32_t ldb2(const uint8_t *base, uint32_t i)
{
    return *reinterpret_cast<const u8x2 *>(base + i);
}
__device__ __forceinline__ void stb2(uint8_t *base, uint32_t i, uint32_t v)
{
    *reinterpret_cast<u8x2 *>(base + i) = (uint16_t)v;
}

// ---------------------------------------------------------------------------
// Land erosion: a land cell with a water 4-neighbour (outside = land) turns
// into water of the given depth, its surface the largest surface among those
// water neighbours, its momenta 0.  Output mask holds 0/1.  Lanes 1..62 store.
constexpr int kInnerStrip = 62;

__global__ __launch_bounds__(256) void erode_kernel(int nx, int ny, int nsx, int nitems,
                                                    const uint8_t *__restrict__ land, const float *__restrict__ Hm,
                                                    const float *__restrict__ eta, const float *__restrict__ hu,
                                                    const float *__restrict__ hv, float depth,
                                                    uint8_t *__restrict__ land_o, float *__restrict__ Hm_o,
                                                    float *__restrict__ eta_o, float *__restrict__ hu_o,
                                                    float *__restrict__ hv_o)
{
    constexpr int R = kRegridRows;
    const int item = wave_item();
    if (item >= nitems) return;
    const int lane = threadIdx.x & 63;
    const int i = (item % nsx) * kInnerStrip - 1 + lane, j0 = (item / nsx) * R;
    const uint32_t ic = (uint32_t)min(max(i, 0), nx - 1);
    const bool col = i >= 0 && i < nx, mine = col && lane >= 1 && lane <= kInnerStrip;

    uint32_t at[R + 2];
    int L[R + 2];
    float e[R + 2], h[R], u[R], v[R];
#pragma unroll
    for (int k = 0; k < R + 2; ++k) {
        at[k] = (uint32_t)min(max(j0 - 1 + k, 0), ny - 1) * (uint32_t)nx + ic;
        L[k] = ldb(land, at[k]);
        e[k] = 0.f;
    }
#pragma unroll
    for (int k = 0; k < R; ++k) { h[k] = ldf(Hm, at[k + 1]); u[k] = v[k] = 0.f; }
    if (eta)
#pragma unroll
        for (int k = 0; k < R + 2; ++k) e[k] = ldf(eta, at[k]);
    if (hu)
#pragma unroll
        for (int k = 0; k < R; ++k) u[k] = ldf(hu, at[k + 1]);
    if (hv)
#pragma unroll
        for (int k = 0; k < R; ++k) v[k] = ldf(hv, at[k + 1]);

    Mask wet[R + 2];
#pragma unroll
    for (int k = 0; k < R + 2; ++k)
        wet[k] = (j0 - 1 + k >= 0 && j0 - 1 + k < ny) ? __builtin_amdgcn_ballot_w64(col && L[k] == 0) : 0;
#pragma unroll
    for (int k = 1; k <= R; ++k) {
        if (j0 + k - 1 >= ny) break;
        const Mask wl = wet[k] << 1, wr = wet[k] >> 1;
        const bool eroded = in(~wet[k] & (wl | wr | wet[k - 1] | wet[k + 1]));
        const float el = lane_left(e[k]), er = lane_right(e[k]);  // shifts need every lane: never under a condition
        float m = -INFINITY;
        m = in(wl) ? fmaxf(m, el) : m;
        m = in(wr) ? fmaxf(m, er) : m;
        m = in(wet[k - 1]) ? fmaxf(m, e[k - 1]) : m;
        m = in(wet[k + 1]) ? fmaxf(m, e[k + 1]) : m;
        if (mine) {
            land_o[at[k]] = (in(wet[k]) || eroded) ? 0 : 1;
            stf(Hm_o, at[k], eroded ? depth : h[k - 1]);
            if (eta) stf(eta_o, at[k], eroded ? m : e[k]);
            if (hu) stf(hu_o, at[k], eroded ? 0.0f : u[k - 1]);
            if (hv) stf(hv_o, at[k], eroded ? 0.0f : v[k - 1]);
        }
    }
}

// ---------------------------------------------------------------------------
// Factor-two refinement of cell fields: generalized-minmod slopes per cell
// (a difference toward land or the outside is 0), evaluated at the four
// sub-cell centres.  The land mask is inherited by the children (field 0
// writes it).
__device__ __forceinline__ float minmod3(float a, float b, float c)
{
    if (a > 0.0f && b > 0.0f && c > 0.0f) return fminf(a, fminf(b, c));
    if (a < 0.0f && b < 0.0f && c < 0.0f) return fmaxf(a, fmaxf(b, c));
    return 0.0f;
}

// item = strip + nsx * (segment of rows) of one field; lanes 1..62 store
__device__ __forceinline__ void refine_cells(int nx, int ny, int strip, int seg, const float *__restrict__ in_f,
                                             const uint8_t *__restrict__ land, float theta, float *__restrict__ out,
                                             uint8_t *__restrict__ land_o)
{
    constexpr int R = kRegridRows;
    const int lane = threadIdx.x & 63;
    const int i = strip * kInnerStrip - 1 + lane, j0 = seg * R;
    const uint32_t ic = (uint32_t)min(max(i, 0), nx - 1);
    const bool col = i >= 0 && i < nx, mine = col && lane >= 1 && lane <= kInnerStrip;

    float c[R + 2];
    int L[R + 2];
#pragma unroll
    for (int k = 0; k < R + 2; ++k) {
        const uint32_t at = (uint32_t)min(max(j0 - 1 + k, 0), ny - 1) * (uint32_t)nx + ic;
        c[k] = ldf(in_f, at);
        L[k] = 0;
        if (land) L[k] = ldb(land, at);
    }
    Mask wet[R + 2];
#pragma unroll
    for (int k = 0; k < R + 2; ++k)
        wet[k] = (j0 - 1 + k >= 0 && j0 - 1 + k < ny) ? __builtin_amdgcn_ballot_w64(col && L[k] == 0) : 0;
#pragma unroll
    for (int k = 1; k <= R; ++k) {
        const int j = j0 + k - 1;
        if (j >= ny) break;
        const Mask w = wet[k];
        const float cl = lane_left(c[k]), cr = lane_right(c[k]);
        const float dl = in(w << 1) ? c[k] - cl : 0.0f;
        const float dr = in(w >> 1) ? cr - c[k] : 0.0f;
        const float ds = in(wet[k - 1]) ? c[k] - c[k - 1] : 0.0f;
        const float dn = in(wet[k + 1]) ? c[k + 1] - c[k] : 0.0f;
        const bool water = in(w);
        const float sx = water ? minmod3(theta * dl, 0.5f * (dl + dr), theta * dr) : 0.0f;
        const float sy = water ? minmod3(theta * ds, 0.5f * (ds + dn), theta * dn) : 0.0f;
        if (mine) {
            const uint32_t lo = (uint32_t)(2 * j) * (2 * (uint32_t)nx) + 2 * (uint32_t)i, hi = lo + 2 * (uint32_t)nx;
            stf2(out, lo, c[k] + -0.25f * sx + -0.25f * sy, c[k] + 0.25f * sx + -0.25f * sy);
            stf2(out, hi, c[k] + -0.25f * sx + 0.25f * sy, c[k] + 0.25f * sx + 0.25f * sy);
            if (land_o) {
                const uint32_t b = water ? 0u : 0x0101u;
                stb2(land_o, lo, b);
                stb2(land_o, hi, b);
            }
        }
    }
}

// Corner depths at the refined intersections: the bilinear surface of each
// coarse cell at its corners, edge midpoints and centre.  Lanes 0..62 store
// their corner and the midpoint to its right, on their row and between it and
// the next.
constexpr int kCornerStrip = 63;

__device__ __forceinline__ void refine_corners(int nx, int ny, int strip, int seg, const float *__restrict__ Hc,
                                               float *__restrict__ out)
{
    constexpr int R = kRegridRows;
    const int lane = threadIdx.x & 63;
    const int i = strip * kCornerStrip + lane, j0 = seg * R;
    const uint32_t ic = (uint32_t)min(i, nx), NX = 2 * (uint32_t)nx + 1;
    const bool mine = i <= nx && lane < kCornerStrip;

    float c[R + 1];
#pragma unroll
    for (int k = 0; k <= R; ++k) c[k] = ldf(Hc, (uint32_t)min(j0 + k, ny) * ((uint32_t)nx + 1) + ic);
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int j = j0 + k;
        if (j > ny) break;
        const float x0 = c[k] + lane_right(c[k]), x1 = c[k + 1] + lane_right(c[k + 1]);
        const uint32_t lo = (uint32_t)(2 * j) * NX + 2 * (uint32_t)i, hi = lo + NX;
        const float ym = 0.5f * (c[k] + c[k + 1]);
        if (mine && i < nx) {
            stf2(out, lo, c[k], 0.5f * x0);
            if (j < ny) stf2(out, hi, ym, 0.25f * (x0 + x1));
        } else if (mine) {
            stf(out, lo, c[k]);
            if (j < ny) stf(out, hi, ym);
        }
    }
}

// One launch of a refinement or a coarsening: `cells` items (strips fastest,
// then segments of rows, then fields) and behind them the corners' items.
struct RegridItems {
    int cells, sx, sy;     // items, strips and segments of a field
    int corners, cx, cy;   // the same of the corner plane
};

__global__ __launch_bounds__(256) void refine_kernel(int nx, int ny, RegridItems n, const float *__restrict__ in_f,
                                                     const uint8_t *__restrict__ land, float theta,
                                                     float *__restrict__ out, uint8_t *__restrict__ land_o,
                                                     const float *__restrict__ Hc, float *__restrict__ Hc_o)
{
    const int item = wave_item();
    if (item < n.cells) {
        const int row = item / n.sx, f = row / n.sy;
        const int64_t plane = (int64_t)nx * ny;
        refine_cells(nx, ny, item - row * n.sx, row - f * n.sy, in_f + f * plane, land, theta, out + f * 4 * plane,
                     f == 0 ? land_o : nullptr);
    } else if (item - n.cells < n.corners) {
        const int k = item - n.cells, row = k / n.cx;
        refine_corners(nx, ny, k - row * n.cx, row, Hc, Hc_o);
    }
}

// Factor-two coarsening: the average of the water children (all four when
// none is water); a coarse cell is land when all four children are.
__device__ __forceinline__ void coarsen_cells(int nx, int ny, int strip, int seg, const float *__restrict__ in_f,
                                              const uint8_t *__restrict__ land, float *__restrict__ out,
                                              uint8_t *__restrict__ land_o)
{
    constexpr int R = kRegridRows;
    const int cx = nx / 2, cy = ny / 2;
    const int i = strip * 64 + (int)(threadIdx.x & 63), j0 = seg * R;
    const uint32_t ic = (uint32_t)min(i, cx - 1);

    f32x2 a[R], b[R];
    uint32_t La[R], Lb[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const uint32_t at = (uint32_t)(2 * min(j0 + k, cy - 1)) * (uint32_t)nx + 2 * ic;
        a[k] = ldf2(in_f, at);
        b[k] = ldf2(in_f, at + (uint32_t)nx);
        La[k] = Lb[k] = 0;
        if (land) { La[k] = ldb2(land, at); Lb[k] = ldb2(land, at + (uint32_t)nx); }
    }
    if (i >= cx) return;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        if (j0 + k >= cy) break;
        bool w0 = (La[k] & 0xff) == 0, w1 = (La[k] >> 8) == 0, w2 = (Lb[k] & 0xff) == 0, w3 = (Lb[k] >> 8) == 0;
        const bool any = w0 | w1 | w2 | w3;
        w0 |= !any; w1 |= !any; w2 |= !any; w3 |= !any;
        float s = 0.0f;
        s = w0 ? s + a[k].x : s;
        s = w1 ? s + a[k].y : s;
        s = w2 ? s + b[k].x : s;
        s = w3 ? s + b[k].y : s;
        const int n = (int)w0 + (int)w1 + (int)w2 + (int)w3;
        const uint32_t o = (uint32_t)(j0 + k) * (uint32_t)cx + (uint32_t)i;
        stf(out, o, s / (float)n);
        if (land_o) land_o[o] = any ? 0 : 1;
    }
}

__device__ __forceinline__ void coarsen_corners(int nx, int ny, int strip, int seg, const float *__restrict__ Hc,
                                                float *__restrict__ out)
{
    constexpr int R = kRegridRows;
    const int CX = nx / 2 + 1, CY = ny / 2 + 1;
    const int i = strip * 64 + (int)(threadIdx.x & 63), j0 = seg * R;
    float c[R];
#pragma unroll
    for (int k = 0; k < R; ++k)
        c[k] = ldf(Hc, (uint32_t)(2 * min(j0 + k, CY - 1)) * ((uint32_t)nx + 1) + 2 * (uint32_t)min(i, CX - 1));
    if (i >= CX) return;
#pragma unroll
    for (int k = 0; k < R; ++k)
        if (j0 + k < CY) stf(out, (uint32_t)(j0 + k) * (uint32_t)CX + (uint32_t)i, c[k]);
}

__global__ __launch_bounds__(256) void coarsen_kernel(int nx, int ny, RegridItems n, const float *__restrict__ in_f,
                                                      const uint8_t *__restrict__ land, float *__restrict__ out,
                                                      uint8_t *__restrict__ land_o, const float *__restrict__ Hc,
                                                      float *__restrict__ Hc_o)
{
    const int item = wave_item();
    if (item < n.cells) {
        const int row = item / n.sx, f = row / n.sy;
        const int64_t plane = (int64_t)nx * ny;
        coarsen_cells(nx, ny, item - row * n.sx, row - f * n.sy, in_f + f * plane, land, out + f * (plane / 4),
                      f == 0 ? land_o : nullptr);
    } else if (item - n.cells < n.corners) {
        const int k = item - n.cells, row = k / n.cx;
        coarsen_corners(nx, ny, k - row * n.cx, row, Hc, Hc_o);
    }
}

// ---------------------------------------------------------------------------
// State planes out of a domain's frames into dense device planes, and the
// control block's head and CFL slots into pinned host memory, in one launch:
// a read is bound by its calls (a 2-D copy call for each plane and one for the
// control block took 30 us, this 18; 2600 x 900 47 and 23, 4096 x 4096 164 and
// 84).  A wave moves
// kReadRows rows of 128 columns of one plane, two columns a lane.
constexpr int kReadRows = 8, kReadCols = 128;

__global__ __launch_bounds__(256) void read_state_kernel(swe::StateRead q, int nsx, int nsy, int nitems)
{
    const int item = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    if (item > nitems) return;
    if (item == nitems) {  // one wave more: the control block
        constexpr int head = offsetof(swe::Ctrl, wslot) / 4;
        const uint32_t *c = reinterpret_cast<const uint32_t *>(q.ctrl);
        uint32_t *o = reinterpret_cast<uint32_t *>(q.ctrl_out);
        for (int k = lane; k < head; k += 64) o[k] = c[k];
        for (int k = lane; k < 2 * swe::kCflSlots; k += 64)
            q.ctrl_out->wslot[k / swe::kCflSlots][k % swe::kCflSlots][0] =
                q.ctrl->wslot[k / swe::kCflSlots][k % swe::kCflSlots][0];
        return;
    }
    const int row = item / nsx, k = row / nsy, y0 = (row - k * nsy) * kReadRows;
    const int x = (item - row * nsx) * kReadCols + 2 * lane;
    if (x >= q.nx) return;
    const float *src = k == 0 ? q.src[0] : k == 1 ? q.src[1] : q.src[2];
    float *dst = k == 0 ? q.dst[0] : k == 1 ? q.dst[1] : q.dst[2];
    const uint32_t at = (uint32_t)min(x, max(q.nx - 2, 0));  // a lane on the last odd column loads the two before its end
    f32x2 v[kReadRows];
#pragma unroll
    for (int j = 0; j < kReadRows; ++j)
        v[j] = ldf2(src, (uint32_t)min(y0 + j, q.ny - 1) * (uint32_t)q.pitch + at);
#pragma unroll
    for (int j = 0; j < kReadRows; ++j) {
        if (y0 + j >= q.ny) break;
        const uint32_t to = (uint32_t)(y0 + j) * (uint32_t)q.nx + (uint32_t)x;
        if (x + 1 < q.nx) stf2(dst, to, v[j].x, v[j].y);
        else stf(dst, to, at < (uint32_t)x ? v[j].y : v[j].x);
    }
}

constexpr int64_t kPlaneLimit = (int64_t)1 << 32;  // bytes of any one plane

bool plane_ok(int64_t rows, int64_t cols, int64_t elem) { return rows * cols * elem < kPlaneLimit; }

int hip_error(hipError_t e, const char *what)
{
    return set_error(SWE_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

// Calls launch(first field, items) until all fields and, with the first of
// them, the corners are done: one launch unless the number of work items
// would leave 32 bits.
template <class Launch>
int for_field_groups(int32_t n_fields, int64_t sx, int64_t sy, bool corners, int64_t cx, int64_t cy, Launch &&launch)
{
    const int64_t most = std::max<int64_t>(1, ((int64_t)1 << 30) / (sx * sy));  // sx sy <= 2^28: planes below 4 GiB
    for (int64_t f0 = 0; f0 < n_fields || (f0 == 0 && corners); f0 += most) {
        const int64_t nf = std::min<int64_t>(n_fields - f0, most);
        RegridItems n{(int)(nf * sx * sy), (int)sx, (int)sy, 0, (int)cx, (int)cy};
        if (f0 == 0 && corners) n.corners = (int)(cx * cy);
        launch(f0, n);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_error(e, "regrid launch");
    }
    return SWE_OK;
}

}  // namespace

hipError_t swe::launch_read_state(const StateRead &q, hipStream_t s)
{
    const int64_t nsx = div_up(q.nx, kReadCols), nsy = div_up(q.ny, kReadRows), items = nsx * nsy * q.planes;
    hipLaunchKernelGGL(read_state_kernel, dim3((unsigned)div_up(items + 1, 4)), dim3(256), 0, s, q, (int)nsx, (int)nsy,
                       (int)items);
    return hipGetLastError();
}

extern "C" int swe_reconstruct_bathymetry(int32_t nx, int32_t ny, const float *Hm, const uint8_t *land,
                                          int32_t iters, float smooth, float *Hc, float *scratch,
                                          void *hip_stream)
{
    if (nx < 1 || ny < 1) return set_error(SWE_E_ARG, "nx and ny must be >= 1");
    if (!plane_ok(ny + 1, nx + 1, 4)) return set_error(SWE_E_ARG, "corner plane must stay below 4 GiB");
    if (!Hm || !Hc) return set_error(SWE_E_ARG, "Hm and Hc must be device pointers");
    if (iters < 0 || iters > 100000) return set_error(SWE_E_ARG, "iters must be in [0, 100000]");
    if (iters > 0 && !scratch) return set_error(SWE_E_ARG, "scratch is required when iters > 0");
    if (!(smooth >= 0.0f && smooth <= 1.0f)) return set_error(SWE_E_ARG, "smooth must be in [0, 1]");
    hipStream_t s = (hipStream_t)hip_stream;
    // the launches of two rounds each end in Hc; the first takes the initial
    // guess alone when the number of rounds is even
    int launches = iters / 2 + 1, k = 0;
    float *buf[2] = {Hc, scratch}, *cur = buf[(launches - 1) & 1];
    hipError_t e = (iters & 1) ? launch_recon<true, true>(s, nx, ny, Hm, land, nullptr, smooth, cur)
                               : launch_recon<true, false>(s, nx, ny, Hm, land, nullptr, smooth, cur);
    while (e == hipSuccess && ++k < launches) {
        float *nxt = buf[(launches - 1 - k) & 1];
        e = launch_recon<false, true>(s, nx, ny, Hm, land, cur, smooth, nxt);
        cur = nxt;
    }
    if (e != hipSuccess) return hip_error(e, "recon_round_kernel");
    return SWE_OK;
}

// ---------------------------------------------------------------------------
// Allocation-free reconstruction: the corner plane the rounds ping-pong
// through lives in a device array of the library's own instead of caller
// memory.  Each GPU the library runs on holds its own copy of the array
// until the process ends; in host code the array's name is only a stand-in,
// so its device address is looked up once per device (hipGetSymbolAddress,
// with that device current) and only that address is handed to kernels.
// Every round overwrites every corner of the plane it writes, so nothing in
// the array has to start at zero.
// ---------------------------------------------------------------------------
namespace {

constexpr int64_t kStaticScratchFloats = (int64_t)4 << 20;  // 16 MiB: up to 4,194,304 corners
static __device__ __align__(256) float scratch[kStaticScratchFloats];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch_ptr[kMaxDevices] = {};

// device address of this device's copy of `scratch`
int static_scratch(float **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_error(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return set_error(SWE_E_ARG, "device index beyond the static scratch table");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_error(e, "hipGetSymbolAddress(scratch)");
        if (!p) return set_error(SWE_E_HIP, "hipGetSymbolAddress(scratch) returned NULL");
        g_scratch_ptr[dev] = static_cast<float *>(p);
    }
    *out = g_scratch_ptr[dev];
    return SWE_OK;
}

}  // namespace

extern "C" int swe_reconstruct_bathymetry_noalloc(int32_t nx, int32_t ny, const float *Hm, const uint8_t *land,
                                                  int32_t iters, float smooth, float *Hc, void *hip_stream)
{
    if (nx < 1 || ny < 1) return set_error(SWE_E_ARG, "nx and ny must be >= 1");
    if ((int64_t)(nx + 1) * (int64_t)(ny + 1) > kStaticScratchFloats)
        return set_error(SWE_E_ARG, "corner plane larger than the static scratch ((nx+1)(ny+1) <= 4194304)");
    float *scr = nullptr;
    if (iters > 0) {
        const int rc = static_scratch(&scr);
        if (rc != SWE_OK) return rc;
    }
    return swe_reconstruct_bathymetry(nx, ny, Hm, land, iters, smooth, Hc, scr, hip_stream);
}

extern "C" int swe_erode_land(int32_t nx, int32_t ny, const uint8_t *land, const float *Hm, const float *eta,
                              const float *hu, const float *hv, float land_depth, uint8_t *land_out,
                              float *Hm_out, float *eta_out, float *hu_out, float *hv_out, void *hip_stream)
{
    if (nx < 1 || ny < 1) return set_error(SWE_E_ARG, "nx and ny must be >= 1");
    if (!plane_ok(ny, nx, 4)) return set_error(SWE_E_ARG, "cell plane must stay below 4 GiB");
    if (!land || !Hm || !land_out || !Hm_out) return set_error(SWE_E_ARG, "land, Hm and their outputs are required");
    if ((eta == nullptr) != (eta_out == nullptr) || (hu == nullptr) != (hu_out == nullptr) ||
        (hv == nullptr) != (hv_out == nullptr))
        return set_error(SWE_E_ARG, "eta, hu and hv need an output exactly when given");
    if (!std::isfinite(land_depth)) return set_error(SWE_E_ARG, "land_depth must be finite");
    const int64_t nsx = div_up(nx, kInnerStrip), items = nsx * div_up(ny, kRegridRows);
    hipLaunchKernelGGL(erode_kernel, item_grid(items), dim3(256), 0, (hipStream_t)hip_stream, nx, ny, (int)nsx,
                       (int)items, land, Hm, eta, hu, hv, land_depth, land_out, Hm_out, eta_out, hu_out, hv_out);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SWE_OK : hip_error(e, "erode_kernel");
}

extern "C" int swe_refine2(int32_t nx, int32_t ny, int32_t n_fields, const float *fields, const uint8_t *land,
                           float theta, float *fields_out, uint8_t *land_out, const float *Hc, float *Hc_out,
                           void *hip_stream)
{
    if (nx < 1 || ny < 1 || n_fields < 0) return set_error(SWE_E_ARG, "nx, ny >= 1 and n_fields >= 0 required");
    if (!plane_ok(2 * (int64_t)ny + 1, 2 * (int64_t)nx + 1, 4))
        return set_error(SWE_E_ARG, "refined corner plane must stay below 4 GiB");
    if (n_fields > 0 && (!fields || !fields_out)) return set_error(SWE_E_ARG, "fields and fields_out are required");
    if (land_out && (!land || n_fields == 0)) return set_error(SWE_E_ARG, "land_out needs land and at least one field");
    if ((Hc == nullptr) != (Hc_out == nullptr)) return set_error(SWE_E_ARG, "Hc and Hc_out go together");
    if (!(theta >= 1.0f && theta <= 2.0f)) return set_error(SWE_E_ARG, "theta must be in [1, 2]");
    const int64_t plane = (int64_t)nx * ny;
    return for_field_groups(
        n_fields, div_up(nx, kInnerStrip), div_up(ny, kRegridRows), Hc != nullptr, div_up((int64_t)nx + 1, kCornerStrip),
        div_up((int64_t)ny + 1, kRegridRows), [&](int64_t f0, const RegridItems &n) {
            hipLaunchKernelGGL(refine_kernel, item_grid((int64_t)n.cells + n.corners), dim3(256), 0,
                               (hipStream_t)hip_stream, nx, ny, n, fields + f0 * plane, land, theta,
                               fields_out + f0 * 4 * plane, f0 == 0 ? land_out : nullptr, Hc, Hc_out);
        });
}

extern "C" int swe_coarsen2(int32_t nx, int32_t ny, int32_t n_fields, const float *fields, const uint8_t *land,
                            float *fields_out, uint8_t *land_out, const float *Hc, float *Hc_out, void *hip_stream)
{
    if (nx < 2 || ny < 2 || (nx & 1) || (ny & 1) || n_fields < 0)
        return set_error(SWE_E_ARG, "nx and ny must be even and >= 2, n_fields >= 0");
    if (!plane_ok(ny + 1, nx + 1, 4)) return set_error(SWE_E_ARG, "corner plane must stay below 4 GiB");
    if (n_fields > 0 && (!fields || !fields_out)) return set_error(SWE_E_ARG, "fields and fields_out are required");
    if (land_out && (!land || n_fields == 0)) return set_error(SWE_E_ARG, "land_out needs land and at least one field");
    if ((Hc == nullptr) != (Hc_out == nullptr)) return set_error(SWE_E_ARG, "Hc and Hc_out go together");
    const int64_t plane = (int64_t)nx * ny;
    return for_field_groups(
        n_fields, div_up(nx / 2, 64), div_up(ny / 2, kRegridRows), Hc != nullptr, div_up(nx / 2 + 1, 64),
        div_up(ny / 2 + 1, kRegridRows), [&](int64_t f0, const RegridItems &n) {
            hipLaunchKernelGGL(coarsen_kernel, item_grid((int64_t)n.cells + n.corners), dim3(256), 0,
                               (hipStream_t)hip_stream, nx, ny, n, fields + f0 * plane, land,
                               fields_out + f0 * (plane / 4), f0 == 0 ? land_out : nullptr, Hc, Hc_out);
        });
}
