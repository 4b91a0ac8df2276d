// HIP kernels of the CodedReduce hot path for gfx950 (64-wide wavefronts).  Everything here is bandwidth bound (stage 1 with every
// holder's bf16 rows done separately: bound by vector-ALU issue): plain vector multiply-adds, 16-byte coalesced loads, no matrix cores.
//
//   rows_once_kernel, rows_once_team_kernel   CR.Execute step 1: X[b:e]^T (phi(X[b:e] w) - y[b:e]) in ONE pass over X, every row's
//                          contribution formed once for all workers that hold it
//   partial_grads_kernel   the same for every holder separately (the splits that lay out every holder's own work)
//   rows_once_crew_kernel  the same for rows too wide for one workgroup, shared by several
//   wide_residuals_kernel, wide_xt_kernel   rows wider still, and wide rows of small matrices, every row once, in two passes
//   residuals_kernel, xt_residuals_kernel   the same for every holder separately
//   sum_rows_kernel        sums of partial rows (fixed order, so results are reproducible bit for bit)
//   tree_kernel            CR.Execute steps 2-5: every node's message, the nodes of a sub-tree side by side, children folded in LDS
//   encode_kernel          the same for long vectors and large trees: one thread walks a sub-tree, children folded in registers
//   decode_kernel          the master's decode  g = sum_j a_j m_(1,j), optionally followed by w <- w - lr g in the same launch
//   tree_decode_kernel     tree_kernel and decode_kernel in one launch, for short vectors
//   update_kernel          w <- w - lr g
//   measures_kernel        the convergence measures of eq. (6) and (8), from the sums that the launches with the gradient step leave
//
// Rows of d elements start on a 4-byte (fp32) or 2-byte (bf16) boundary whatever d is, so the 16-byte row accesses are declared
// with that alignment; the hardware runs in unaligned-access mode and the compiler emits the same dwordx4 instructions.
// A row is cut into nq = ceil(d / VEC) chunks of VEC columns; when VEC does not divide d the last chunk is moved back to end at
// column d, overlapping its neighbour.  Overlapped columns are then produced twice, from the same operands in the same order,
// and both copies store the same bits; only sums ACROSS columns (the dot product x.w) must count them once.
#include "kernels.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>
#include <iterator>
#include <type_traits>

namespace cr {

namespace {

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));       // four floats of an fp32 row
typedef unsigned u4h __attribute__((ext_vector_type(4), aligned(2)));    // eight bf16 values of a bf16 row
typedef float f4a __attribute__((ext_vector_type(4)));                   // four floats on a 16-byte boundary

// v + (v of the lane that the cross-lane pattern CTRL pairs this lane with, inside its row of 16 lanes)
template <int CTRL> __device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// Sum over the 64 lanes, delivered to every lane.  The four steps inside a row of 16 lanes are adds that read the partner lane
// directly (quad swaps, then the mirrored half-row and row: for a sum a mirror does what an exchange does).  The two steps across
// rows either go through the LDS crossbar (2 adds + 2 LDS operations), or pass lane 15 / lane 31 on to the following rows so
// that lane 63 ends with the total, which is then read into a scalar register (5 vector operations, no LDS round trip).
// Kernels limited by vector-ALU issue (bf16 rows: a widening operation per element on top of the two multiply-adds) take the
// first form, kernels limited by cache bandwidth and latency (fp32 rows) the second.
template <bool VIA_LDS> __device__ __forceinline__ float wave_sum(float v)
{
    v = dpp_add<0xB1>(v);      // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);      // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v);     // row_half_mirror
    v = dpp_add<0x140>(v);     // row_mirror
    if constexpr (VIA_LDS) {
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        return v;
    } else {
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x142, 0xa, 0xf, false));   // row_bcast:15 into rows 1 and 3
        v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x143, 0xc, 0xf, false));   // row_bcast:31 into rows 2 and 3
        return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
    }
}

// The same for four rows at once, at less than half the vector instructions: a transposing butterfly.  After the first two steps
// (lane pairs, then pairs of pairs, each lane keeping the row its position selects and handing the other to its partner) lane l
// holds the sum over its quad of row l & 3; two rotations inside the row of 16 lanes and two exchanges across rows finish the sums,
// and lanes 0..3 hold the four totals.  13 vector operations, 2 LDS exchanges and 4 lane reads for four rows, where four single
// sums take about 44.
// wave_sum4_lanes leaves the totals in the lanes (lane l holds the total of row l & 3); wave_sum4 reads them into scalars.
__device__ __forceinline__ float wave_sum4_lanes(const float (&s)[4])
{
    const unsigned lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const bool b0 = lane & 1u, b1 = lane & 2u;
    // lanes with b0 = 0 keep rows 0 and 2, the others rows 1 and 3
    float t01 = (b0 ? s[1] : s[0]) + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(b0 ? s[0] : s[1]), 0xB1, 0xf, 0xf, false));
    float t23 = (b0 ? s[3] : s[2]) + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(b0 ? s[2] : s[3]), 0xB1, 0xf, 0xf, false));
    // lanes with b1 = 0 keep rows 0/1, the others rows 2/3
    float u = (b1 ? t23 : t01) + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(b1 ? t01 : t23), 0x4E, 0xf, 0xf, false));
    u += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(u), 0x124, 0xf, 0xf, false));      // row_ror:4
    u += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(u), 0x128, 0xf, 0xf, false));      // row_ror:8
    u += __shfl_xor(u, 16, 64);
    u += __shfl_xor(u, 32, 64);
    return u;
}
__device__ __forceinline__ void wave_sum4(const float (&s)[4], float (&out)[4])
{
    const float u = wave_sum4_lanes(s);
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(u), r));
}

// 1 / (1 + e^-z) from the hardware exponential and reciprocal (each good to about one unit in the last place); it saturates to
// 0 and 1 for large |z| without special cases
__device__ __forceinline__ float sigmoid(float z) { return __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

// element offset of chunk q inside a row (a chunk index past the row is sent to the last chunk)
template <int VEC> __device__ __forceinline__ int chunk_offset(int q, int nq, int d)
{
    return q < nq - 1 ? q * VEC : d - VEC;
}
// does element v of chunk q belong to it alone (not to the overlap with the chunk before, not past the row)?
template <int VEC> __device__ __forceinline__ bool chunk_owns(int q, int v, int nq, int d)
{
    return q < nq - 1 || (q == nq - 1 && d - VEC + v >= (nq - 1) * VEC);
}

// Element v of chunk q if it belongs to it alone.  The dot products meet the others, which another lane counts, with weights of zero, which
// is right for every number.  Infinity times zero is none: where a logistic dot product is not a number it is formed once more from these, by
// the run where a wavefront forms its rows alone, by the step where a workgroup shares them (1 200 x 100, 20 steps 223 us with and without,
// launches of 8 us up to 0.2 us more, 252 000 x 4 096 602 / 604).  The kernels that do every holder's rows separately leave it at the weights.
template <int VEC> __device__ __forceinline__ float counted(float x, int q, int v, int nq, int d) { return chunk_owns<VEC>(q, v, nq, d) ? x : 0.f; }

// ---- how a chunk of a row of X is fetched and widened to fp32 -------------------------------------------------
// load(row, e): the chunk at element e of the row that starts at `row` (a wave-uniform pointer; e differs per lane);
// load_once: the same for rows nobody else reads, with the non-temporal hint, so that they stream past the caches
template <int XD, int VEC> struct Chunk;
template <int XD> __device__ __forceinline__ const void *row_ptr(const void *X, int64_t row, int d)
{
    return static_cast<const char *>(X) + row * d * (XD == 1 ? 2 : 4);
}

template <> struct Chunk<0, 4> {
    using raw_t = f4u;
    static __device__ __forceinline__ raw_t load(const void *row, unsigned e) { return *reinterpret_cast<const f4u *>(static_cast<const char *>(row) + e * 4u); }
    static __device__ __forceinline__ raw_t load_once(const void *row, unsigned e) { return __builtin_nontemporal_load(reinterpret_cast<const f4u *>(static_cast<const char *>(row) + e * 4u)); }
    static __device__ __forceinline__ void widen(const raw_t &r, float (&v)[4]) { v[0] = r.x; v[1] = r.y; v[2] = r.z; v[3] = r.w; }
};
template <> struct Chunk<1, 8> {
    using raw_t = u4h;
    static __device__ __forceinline__ raw_t load(const void *row, unsigned e) { return *reinterpret_cast<const u4h *>(static_cast<const char *>(row) + e * 2u); }
    static __device__ __forceinline__ raw_t load_once(const void *row, unsigned e) { return __builtin_nontemporal_load(reinterpret_cast<const u4h *>(static_cast<const char *>(row) + e * 2u)); }
    static __device__ __forceinline__ void widen(const raw_t &r, float (&v)[8])
    {
        v[0] = __uint_as_float(r.x << 16); v[1] = __uint_as_float(r.x & 0xffff0000u);
        v[2] = __uint_as_float(r.y << 16); v[3] = __uint_as_float(r.y & 0xffff0000u);
        v[4] = __uint_as_float(r.z << 16); v[5] = __uint_as_float(r.z & 0xffff0000u);
        v[6] = __uint_as_float(r.w << 16); v[7] = __uint_as_float(r.w & 0xffff0000u);
    }
};
template <> struct Chunk<0, 1> {      // rows shorter than one wide chunk
    using raw_t = float;
    static __device__ __forceinline__ raw_t load(const void *row, unsigned e) { return *reinterpret_cast<const float *>(static_cast<const char *>(row) + e * 4u); }
    static __device__ __forceinline__ raw_t load_once(const void *row, unsigned e) { return __builtin_nontemporal_load(reinterpret_cast<const float *>(static_cast<const char *>(row) + e * 4u)); }
    static __device__ __forceinline__ void widen(const raw_t &r, float (&v)[1]) { v[0] = r; }
};
template <> struct Chunk<1, 1> {
    using raw_t = uint16_t;
    static __device__ __forceinline__ raw_t load(const void *row, unsigned e) { return *reinterpret_cast<const uint16_t *>(static_cast<const char *>(row) + e * 2u); }
    static __device__ __forceinline__ raw_t load_once(const void *row, unsigned e) { return __builtin_nontemporal_load(reinterpret_cast<const uint16_t *>(static_cast<const char *>(row) + e * 2u)); }
    static __device__ __forceinline__ void widen(const raw_t &r, float (&v)[1]) { v[0] = __uint_as_float(static_cast<uint32_t>(r) << 16); }
};

template <typename T> __device__ __forceinline__ T *at_byte(T *p, unsigned bytes)
{
    return reinterpret_cast<T *>(reinterpret_cast<std::conditional_t<std::is_const_v<T>, const char, char> *>(p) + bytes);
}

// VEC consecutive floats of an fp32 row (slab gradients, piece partials, messages)
template <int VEC> __device__ __forceinline__ void load_row(const float *src, float (&v)[VEC])
{
    if constexpr (VEC % 4 == 0) {
#pragma unroll
        for (int i = 0; i < VEC; i += 4) { const f4u t = *reinterpret_cast<const f4u *>(src + i); v[i] = t.x; v[i + 1] = t.y; v[i + 2] = t.z; v[i + 3] = t.w; }
    } else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = src[i];
    }
}
template <int VEC> __device__ __forceinline__ void load_row_nt(const float *src, float (&v)[VEC])
{
    if constexpr (VEC % 4 == 0) {
#pragma unroll
        for (int i = 0; i < VEC; i += 4) { const f4u t = __builtin_nontemporal_load(reinterpret_cast<const f4u *>(src + i)); v[i] = t.x; v[i + 1] = t.y; v[i + 2] = t.z; v[i + 3] = t.w; }
    } else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) v[i] = __builtin_nontemporal_load(src + i);
    }
}
template <int VEC> __device__ __forceinline__ void store_row(float *dst, const float (&v)[VEC])
{
    if constexpr (VEC % 4 == 0) {
#pragma unroll
        for (int i = 0; i < VEC; i += 4) { f4u t; t.x = v[i]; t.y = v[i + 1]; t.z = v[i + 2]; t.w = v[i + 3]; *reinterpret_cast<f4u *>(dst + i) = t; }
    } else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) dst[i] = v[i];
    }
}
template <int VEC> __device__ __forceinline__ void store_row_nt(float *dst, const float (&v)[VEC])
{
    if constexpr (VEC % 4 == 0) {
#pragma unroll
        for (int i = 0; i < VEC; i += 4) { f4u t; t.x = v[i]; t.y = v[i + 1]; t.z = v[i + 2]; t.w = v[i + 3]; __builtin_nontemporal_store(t, reinterpret_cast<f4u *>(dst + i)); }
    } else {
#pragma unroll
        for (int i = 0; i < VEC; ++i) __builtin_nontemporal_store(v[i], dst + i);
    }
}

// ---- stage 1 ------------------------------------------------------------------------------------------------------
// A team of TS threads owns whole rows: thread t holds chunks t, t+TS, ... (K of them, VEC columns each) of every row it
// works on, so a row is fetched once, used for the dot product x.w, kept in registers, and used again for the rank-1 update
// acc += (phi(x.w) - y) x.  R rows are in flight per step.  The dot is reduced inside the wavefront and, for teams of several
// wavefronts, through LDS (double buffered: one barrier per step).  Each piece ends with one d-float store of the accumulators.
template <int XD, int VEC, int TS, int K, int R, bool LOGISTIC, bool BUF = false>
__global__ void __launch_bounds__((TS < 256 ? 256 : TS))
partial_grads_kernel(const void *__restrict__ X, const float *__restrict__ y, const float *__restrict__ w,
                     const DevPiece *__restrict__ pieces, const int32_t *__restrict__ team_piece_begin, int num_teams,
                     float *__restrict__ rows, int d, int nq)
{
    using C = Chunk<XD, VEC>;
    using raw_t = typename C::raw_t;
    constexpr int BLOCK = TS < 256 ? 256 : TS;
    constexpr int WAVES = TS / 64;
    const int tl = threadIdx.x % TS;
    // the team index is the same for every lane of a wavefront: keep it (and all that derives from it) in scalar registers
    const int team = __builtin_amdgcn_readfirstlane(blockIdx.x * (BLOCK / TS) + threadIdx.x / TS);
    __shared__ float red[2][R][WAVES];
    if (team >= num_teams) return;   // whole teams only; teams of several wavefronts span the block, so barriers stay uniform

    // K = ceil(nq / TS): only the last chunk of a thread can fall outside the row.  Such a lane re-reads the row's last chunk
    // (so every load is unconditional) with zero weights, and never stores its accumulator.
    unsigned off[K];
    float wv[K][VEC];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = tl + k * TS;
        off[k] = chunk_offset<VEC>(q, nq, d);
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const float t = w[off[k] + v];               // always inside the row; masked after the load
            wv[k][v] = chunk_owns<VEC>(q, v, nq, d) ? t : 0.f;
        }
    }

    const int lane3 = tl & 3;
    const int pb = team_piece_begin[team], pe = team_piece_begin[team + 1];
    int buf = 0;
    for (int p = pb; p < pe; ++p) {
        const DevPiece pc = pieces[p];
        float acc[K][VEC];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[k][v] = 0.f;

        // BUF (chosen by the host where every row starts on a 4-byte boundary and every piece has fewer than 2^31 bytes): the
        // piece's rows as a buffer -- base, size in bytes, plain 32-bit words
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(row_ptr<XD>(X, pc.row_begin, d)), 0,
                                                                                 BUF ? pc.nrows * d * (XD == 1 ? 2 : 4) : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(y + pc.row_begin), 0, BUF ? pc.nrows * 4 : 0, 0x00020000);
        for (int r0 = 0; r0 < pc.nrows; r0 += R) {
            raw_t xr[R][K];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int rr = min(r0 + r, pc.nrows - 1);          // rows past the end re-read the last row; their residual is zeroed
                const void *row = row_ptr<XD>(X, pc.row_begin + rr, d);
                if constexpr (BUF) {
                    // bf16 rows (bound by vector-ALU issue): a buffer load takes the piece's base and the row's offset as scalars
                    // and the lane's offset as it is, where a global load costs a 64-bit vector add per load
                    const unsigned soff = static_cast<unsigned>(rr) * static_cast<unsigned>(d) * (XD == 1 ? 2u : 4u);
#pragma unroll
                    for (int k = 0; k < K; ++k)
                        xr[r][k] = __builtin_bit_cast(raw_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off[k] * (XD == 1 ? 2u : 4u), soff, 0));
                } else if (XD == 1 || pc.shared) {
                    // fp32 rows that other holders read too are left in the L2; bf16 rows always are (that path is bound by the
                    // vector ALUs, and a second copy of its loop costs more than streaming gains)
#pragma unroll
                    for (int k = 0; k < K; ++k) xr[r][k] = C::load(row, off[k]);
                } else {
                    asm volatile("; rows read once" ::: "memory");   // (the markers keep the two kinds of load from being merged into one)
#pragma unroll
                    for (int k = 0; k < K; ++k) xr[r][k] = C::load_once(row, off[k]);
                    asm volatile("; rows read once" ::: "memory");
                }
            }
            float pd[R], res_of[R];
            if constexpr (XD == 1 && R % 4 == 0) {
                // bf16 rows are bound by vector-ALU issue: the cross-lane sums of four rows are taken together
#pragma unroll
                for (int r0b = 0; r0b < R; r0b += 4) {
                    float s4[4], t4[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float s = 0.f;
#pragma unroll
                        for (int k = 0; k < K; ++k) {
                            float xv[VEC];
                            C::widen(xr[r0b + r][k], xv);
#pragma unroll
                            for (int v = 0; v < VEC; ++v) s = fmaf(xv[v], wv[k][v], s);
                        }
                        s4[r] = s;
                    }
                    if constexpr (BUF && WAVES == 1) {
                        // the residuals of the four rows in one go, in the lanes that hold the totals: lane l has the target of row
                        // l & 3 (one 4-byte buffer load per lane; past the piece's end it returns 0 and the row counts for nothing)
                        const float u = wave_sum4_lanes(s4);
                        const float yv = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc_y, lane3 * 4, (r0 + r0b) * 4, 0));
                        const float ph = LOGISTIC ? sigmoid(u) : u;
                        const float rv = lane3 < pc.nrows - (r0 + r0b) ? ph - yv : 0.f;
#pragma unroll
                        for (int r = 0; r < 4; ++r) res_of[r0b + r] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(rv), r));
                    } else {
                        wave_sum4(s4, t4);
#pragma unroll
                        for (int r = 0; r < 4; ++r) pd[r0b + r] = t4[r];
                    }
                }
            } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float s = 0.f;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    float xv[VEC];
                    C::widen(xr[r][k], xv);
#pragma unroll
                    for (int v = 0; v < VEC; ++v) s = fmaf(xv[v], wv[k][v], s);
                }
                pd[r] = wave_sum<XD == 1>(s);
            }
            }
            if constexpr (WAVES > 1) {
                const int wave = tl / 64;
                if ((tl & 63) == 0) {
#pragma unroll
                    for (int r = 0; r < R; ++r) red[buf][r][wave] = pd[r];
                }
                __syncthreads();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float s = 0.f;
#pragma unroll
                    for (int wv_i = 0; wv_i < WAVES; ++wv_i) s += red[buf][r][wv_i];
                    pd[r] = s;
                }
                buf ^= 1;
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int rr = r0 + r;
                float res;
                if constexpr (BUF && XD == 1 && R % 4 == 0 && WAVES == 1) res = res_of[r];
                else {
                    const float yy = y[pc.row_begin + min(rr, pc.nrows - 1)];
                    const float z = pd[r];
                    const float ph = LOGISTIC ? sigmoid(z) : z;
                    res = (rr < pc.nrows) ? ph - yy : 0.f;
                }
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    float xv[VEC];
                    C::widen(xr[r][k], xv);
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[k][v] = fmaf(res, xv[v], acc[k][v]);
                }
            }
        }
        float *out = rows + static_cast<int64_t>(pc.out_row) * d;
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (tl + k * TS < nq) store_row<VEC>(out + off[k], acc[k]);
    }
}

// ---- stage 1, every row once ------------------------------------------------------------------------------------------
// All holders of a row need the same thing of it, (phi(x.w) - y) x, so here it is formed once.  A *run* is a contiguous range of
// rows that no slab begins or ends inside; its gradient goes to every row of the output table its destination list names: straight
// into the slabs that consist of just this run, and into a partial row where larger slabs are summed from several runs
// (sum_rows_kernel).  A workgroup owns one contiguous *part* of X -- in the default split the chip's compute units take one or two
// parts each, so X is read as a few hundred long sequential streams with one wave of workgroups and few partial rows.
// What bounds it is the read of X (a plain streaming read: 7.06 TB/s).  One workgroup per compute unit for rows that a whole workgroup
// shares: 252 000 x 4 096 and 100 000 x 10 000 fp32 7.0 and 6.9 TB/s.  It is slower where the parts' starts lie a large power of two
// apart (196 608 x 4 096, parts of 12 MB: 6.25 with 256 workgroups, 6.80 with 512, 6.72 with 768; x 8 192 bf16 6.26, 6.59, 6.47) and
// the same where they do not (80 530 x 10 000: 6.32, 6.36, 6.28).  Rows of at most 256 chunks, one row per wavefront or less, get two:
// 805 306 x 1 000 fp32 6.45, 6.77, 6.87, 1 572 864 x 1 024 bf16 5.83, 6.77, 6.85.
// The rows of the next step are loaded before the current step is computed (two register sets).
// NT: rows fetched with the non-temporal hint, for matrices larger than the last-level cache.

// The plan's tables are written before the launch: read through the scalar cache, whatever the kernel stores meanwhile.
template <typename T> using table_t = const __attribute__((address_space(4))) T *;
template <typename T> __device__ __forceinline__ table_t<T> table(const T *p) { return (table_t<T>)(p); }
struct Run { int64_t row_begin; int nrows, dst_begin, dst_end; };
__device__ __forceinline__ Run read_run(table_t<DevRun> r) { return {r->row_begin, r->nrows, r->dst_begin, r->dst_end}; }

// Sums over rows are kept in fp64 and rounded once per run; only the R <= 4 rows that a thread has in hand in one step are added in
// fp32 first, which leaves one widening and one fp64 add per R rows.  (fp32 sums folded every 512 rows take the same registers and
// were further from the exact slabs: 100 000 x 20 480 bf16 2.5e-7 against 0.7e-7.)
template <int VEC, int R> __device__ __forceinline__ void add_rows(double (&acc)[VEC], const float (&res)[R], const float (&xv)[R][VEC])
{
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        if constexpr (R == 1) {
            acc[v] = fma(static_cast<double>(res[0]), static_cast<double>(xv[0][v]), acc[v]);
        } else {
            float t = res[0] * xv[0][v];
#pragma unroll
            for (int r = 1; r < R; ++r) t = fmaf(res[r], xv[r][v], t);
            acc[v] += static_cast<double>(t);
        }
    }
}

// phi(z) - y; the choice is the same for the whole launch
__device__ __forceinline__ float residual(float z, float y, int logistic) { return (logistic ? sigmoid(z) : z) - y; }

// Sum over aligned groups of LPR lanes, delivered to every lane of the group, in vector operations only (no LDS round trip).
template <int LPR> __device__ __forceinline__ float group_sum(float v)
{
    if constexpr (LPR >= 2) v = dpp_add<0xB1>(v);       // quad_perm [1,0,3,2]
    if constexpr (LPR >= 4) v = dpp_add<0x4E>(v);       // quad_perm [2,3,0,1]
    if constexpr (LPR >= 8) v = dpp_add<0x141>(v);      // row_half_mirror
    if constexpr (LPR >= 16) v = dpp_add<0x140>(v);     // row_mirror
    if constexpr (LPR >= 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false);
        v = __int_as_float(r[0]) + __int_as_float(r[1]);
    }
    if constexpr (LPR >= 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
        v = __int_as_float(r[0]) + __int_as_float(r[1]);
    }
    return v;
}

// Rows of at most 256 chunks.  LPR lanes share a row (64 / LPR rows side by side in a wavefront), lane t of them holding chunks t,
// t + LPR, ... (K > 1 only with LPR = 64); a wavefront takes R such sets of rows per step.  No barrier until the sums of a run are
// done; then the accumulators of the whole workgroup meet in LDS, are added up and rounded.
template <int XD, int VEC, int LPR, int K, int R, int WAVES, bool NT>
__global__ void __launch_bounds__(WAVES * 64)
rows_once_kernel(const void *__restrict__ X, const float *__restrict__ y, const float *__restrict__ w, const DevRun *__restrict__ parts,
                 const DevRun *__restrict__ runs, const int32_t *__restrict__ dst, float *__restrict__ rows, int d, int nq, int logistic)
{
    static_assert(K == 1 || LPR == 64, "several chunks per lane only for rows of more than 64 chunks");
    using C = Chunk<XD, VEC>;
    constexpr int RPW = 64 / LPR, STEP = WAVES * R * RPW, THREADS = WAVES * 64;
    // SETS sets of COLS accumulators each; where there are fewer columns than threads, GROUPS threads share a column
    constexpr int SETS = WAVES * RPW, COLS = K * LPR * VEC, GROUPS = COLS < THREADS ? THREADS / COLS : 1;
    __shared__ __align__(16) double comb[SETS][COLS];
    __shared__ double comb2[GROUPS > 1 ? GROUPS : 1][GROUPS > 1 ? COLS : 1];
    const int lane = threadIdx.x & 63, sub = lane / LPR, tl = lane % LPR;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const table_t<DevRun> part = table(parts) + blockIdx.x;
    const int more = part->more_end;
    int next = part->more_begin;
    Run run = read_run(part);

    unsigned off[K];                                     // first element of the lane's chunks
    float wv[K][VEC];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = tl + k * LPR;
        off[k] = chunk_offset<VEC>(q, nq, d);
        load_row<VEC>(w + off[k], wv[k]);
#pragma unroll
        for (int v = 0; v < VEC; ++v) wv[k][v] = chunk_owns<VEC>(q, v, nq, d) ? wv[k][v] : 0.f;
    }

    struct Step {
        typename C::raw_t x[R][K];
        float yy[R];
    };
    for (;;) {
        const void *base = row_ptr<XD>(X, run.row_begin, d);
        const float *yb = y + run.row_begin;
        const int n = run.nrows;
        double acc[K][VEC];
        // rows past the end of the run re-read its last row; they count for nothing
        auto load = [&](Step &s, int r0) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int first = min(r0 + (wave * R + r) * RPW, n - 1);
                const void *row = row_ptr<XD>(base, first, d);
                const int mine = RPW == 1 ? first : min(first + sub, n - 1);
                const unsigned rel = RPW == 1 ? 0u : static_cast<unsigned>(mine - first) * static_cast<unsigned>(d);
                s.yy[r] = yb[mine];
#pragma unroll
                for (int k = 0; k < K; ++k) s.x[r][k] = NT ? C::load_once(row, rel + off[k]) : C::load(row, rel + off[k]);
            }
        };
        auto compute = [&](const Step &s, int r0, auto only_counted) {
            float z[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float t = 0.f;
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    float xv[VEC];
                    C::widen(s.x[r][k], xv);
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
                        t = fmaf(decltype(only_counted)::value ? counted<VEC>(xv[v], tl + k * LPR, v, nq, d) : xv[v], wv[k][v], t);
                }
                z[r] = group_sum<LPR>(t);
            }
            float res[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int at = r0 + (wave * R + r) * RPW + (RPW == 1 ? 0 : sub);
                res[r] = at < n ? residual(z[r], s.yy[r], logistic) : 0.f;
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
                float xv[R][VEC];
#pragma unroll
                for (int r = 0; r < R; ++r) C::widen(s.x[r][k], xv[r]);
                add_rows<VEC, R>(acc[k], res, xv);
            }
        };
        auto store = [&] {
            __syncthreads();                             // the sums stored before these have been read
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int v = 0; v < VEC; ++v) comb[wave * RPW + sub][(k * LPR + tl) * VEC + v] = acc[k][v];
            __syncthreads();
            auto put = [&](int c, double t) {
                const float out = static_cast<float>(t);
                const int col = chunk_offset<VEC>(c / VEC, nq, d) + c % VEC;
                for (int j = run.dst_begin; j < run.dst_end; ++j) rows[static_cast<int64_t>(table(dst)[j]) * d + col] = out;
            };
            if constexpr (GROUPS > 1) {
                const int c = threadIdx.x % COLS, g = threadIdx.x / COLS;
                double t = 0.0;
#pragma unroll
                for (int i = 0; i < (SETS + GROUPS - 1) / GROUPS; ++i)
                    if (g + i * GROUPS < SETS) t += comb[g + i * GROUPS][c];
                comb2[g][c] = t;
                __syncthreads();
                if (g == 0 && c < nq * VEC) {
#pragma unroll
                    for (int i = 1; i < GROUPS; ++i) t += comb2[i][c];
                    put(c, t);
                }
            } else {
                for (int c = threadIdx.x; c < nq * VEC; c += THREADS) {
                    double t = 0.0;
#pragma unroll
                    for (int i = 0; i < SETS; ++i) t += comb[i][c];
                    put(c, t);
                }
            }
        };
        auto form = [&](auto only_counted) {
#pragma unroll
            for (int k = 0; k < K; ++k)
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[k][v] = 0.0;
            Step a, b;
            load(a, 0);
            for (int r0 = 0;;) {
                load(b, r0 + STEP);
                compute(a, r0, only_counted);
                if ((r0 += STEP) >= n) break;
                load(a, r0 + STEP);
                compute(b, r0, only_counted);
                if ((r0 += STEP) >= n) break;
            }
        };
        form(std::false_type{});
        // see counted(): a dot product that is not a number leaves no sum of its lane one
        if (__builtin_expect(logistic && !__all(acc[0][0] == acc[0][0]), 0)) form(std::true_type{});
        store();
        if (next >= more) break;
        run = read_run(table(runs) + next++);
    }
}

// Wider rows: the TS threads of the workgroup share every row, thread t holding chunks t, t + TS, ..., R rows per step.  One barrier
// per step exchanges the wavefronts' parts of the dot products (double buffered in LDS).  PF: the next step's rows are loaded before
// the current step is computed; beyond 9 chunks per thread the second register set costs more than it hides (a row is then long
// enough: 12 chunks, 24576 columns, 3.2 GB: 497 us without, 604 with it).
// WL: the weights are in LDS, every thread's in slots of its own, which leaves the registers for rows half as wide again, 34 816 fp32 or
// 36 864 bf16 columns, that took two passes (stage 1 in us, two passes / this: 6 000 x 32 768 fp32 245 / 133, 3 000 x 30 001 fp32 115 / 70,
// 10 000 x 36 864 bf16 225 / 141, 4 000 x 25 000 bf16 68 / 38).  Up to 12 fp32 chunks per thread it gains nothing, not with the next
// row's loads ahead either (3 000 x 24 000: 56.9 without, 58.7 with both).  The widest of these (17 fp32 or 9 bf16 chunks) use all 256
// registers and keep 28 bytes per lane in scratch: 10 000 x 36 864 bf16 takes 1.35 times a plain read of it.
template <int XD, int VEC, int TS, int K, int R, bool PF, bool WL, bool NT>
__global__ void __launch_bounds__(TS)
rows_once_team_kernel(const void *__restrict__ X, const float *__restrict__ y, const float *__restrict__ w, const DevRun *__restrict__ parts,
                      const DevRun *__restrict__ runs, const int32_t *__restrict__ dst, float *__restrict__ rows, int d, int nq, int logistic)
{
    using C = Chunk<XD, VEC>;
    constexpr int WAVES = TS / 64;
    __shared__ float red[2][R][WAVES];
    const int tl = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const table_t<DevRun> part = table(parts) + blockIdx.x;
    const int more = part->more_end;
    int next = part->more_begin;
    Run run = read_run(part);

    // only a thread's last chunk can be the row's last one or past it: the others lie k * TS chunks after the first
    constexpr unsigned kElem = XD == 1 ? 2 : 4;
    const unsigned off = tl * VEC, off_last = chunk_offset<VEC>(tl + (K - 1) * TS, nq, d);
    float wv[WL ? 1 : K][VEC];
    __shared__ f4a wl[WL ? K : 1][WL ? VEC / 4 : 1][WL ? TS : 1];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = tl + k * TS;
        float (&t)[VEC] = wv[WL ? 0 : k];
        load_row<VEC>(w + (k < K - 1 ? k * TS * VEC + off : off_last), t);
#pragma unroll
        for (int v = 0; v < VEC; ++v) t[v] = chunk_owns<VEC>(q, v, nq, d) ? t[v] : 0.f;
        if constexpr (WL)
#pragma unroll
            for (int i = 0; i < VEC / 4; ++i) wl[k][i][tl] = f4a{t[4 * i], t[4 * i + 1], t[4 * i + 2], t[4 * i + 3]};
    }

    const bool ragged = logistic && d != K * TS * VEC;   // elements that no lane counts, or two have: see counted()
    struct Step {
        typename C::raw_t x[R][K];
        float yy[R];
    };
    int buf = 0;
    for (;;) {
        const void *base = row_ptr<XD>(X, run.row_begin, d);
        const float *yb = y + run.row_begin;
        const int n = run.nrows;
        double acc[K][VEC];
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[k][v] = 0.0;
        auto load = [&](Step &s, int r0) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int at = min(r0 + r, n - 1);
                const void *row = row_ptr<XD>(base, at, d);
                s.yy[r] = yb[at];
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const void *from = static_cast<const char *>(row) + (k < K - 1 ? k * TS * VEC * kElem : 0u);
                    const unsigned e = k < K - 1 ? off : off_last;
                    s.x[r][k] = NT ? C::load_once(from, e) : C::load(from, e);
                }
            }
        };
        // the wavefronts' parts of the dot products of a step go to LDS
        auto dots = [&](const Step &s, auto only_counted) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float t[2] = {0.f, 0.f};                 // two chains: a multiply-add need not wait for the one before it
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    float xv[VEC];
                    C::widen(s.x[r][k], xv);
                    if (decltype(only_counted)::value && k == K - 1)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) xv[v] = counted<VEC>(xv[v], tl + k * TS, v, nq, d);
                    if constexpr (WL) {
#pragma unroll
                        for (int i = 0; i < VEC / 4; ++i) {
                            const f4a wt = wl[k][i][tl];
                            t[k & 1] = fmaf(xv[4 * i], wt.x, t[k & 1]);
                            t[k & 1] = fmaf(xv[4 * i + 1], wt.y, t[k & 1]);
                            t[k & 1] = fmaf(xv[4 * i + 2], wt.z, t[k & 1]);
                            t[k & 1] = fmaf(xv[4 * i + 3], wt.w, t[k & 1]);
                        }
                    } else {
#pragma unroll
                        for (int v = 0; v < VEC; ++v) t[k & 1] = fmaf(xv[v], wv[k][v], t[k & 1]);
                    }
                }
                const float dot = group_sum<64>(t[0] + t[1]);
                if ((tl & 63) == 0) red[buf][r][wave] = dot;
            }
            __syncthreads();
        };
        auto compute = [&](const Step &s, int r0) {
            dots(s, std::false_type{});
            float z[R];
            auto sums = [&] {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    z[r] = 0.f;
#pragma unroll
                    for (int i = 0; i < WAVES; ++i) z[r] += red[buf][r][i];
                }
            };
            sums();
            if (ragged) {
                float finite = 0.f;                      // the same for all threads
#pragma unroll
                for (int r = 0; r < R; ++r) finite = fmaf(z[r], 0.f, finite);
                if (__builtin_expect(__builtin_amdgcn_readfirstlane(finite != 0.f), 0)) {
                    __syncthreads();                     // the sums have been read
                    dots(s, std::true_type{});
                    sums();
                }
            }
            float res[R];
#pragma unroll
            for (int r = 0; r < R; ++r) res[r] = r0 + r < n ? residual(z[r], s.yy[r], logistic) : 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                float xv[R][VEC];
#pragma unroll
                for (int r = 0; r < R; ++r) C::widen(s.x[r][k], xv[r]);
                add_rows<VEC, R>(acc[k], res, xv);
            }
            buf ^= 1;
        };
        Step a, b;
        if constexpr (PF) load(a, 0);
        for (int r0 = 0;;) {
            if constexpr (PF) load(b, r0 + R);
            else load(a, r0);
            compute(a, r0);
            if ((r0 += R) >= n) break;
            if constexpr (PF) {
                load(a, r0 + R);
                compute(b, r0);
                if ((r0 += R) >= n) break;
            }
        }
        for (int j = run.dst_begin; j < run.dst_end; ++j) {
            float *out = rows + static_cast<int64_t>(table(dst)[j]) * d;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                float sum[VEC];
#pragma unroll
                for (int v = 0; v < VEC; ++v) sum[v] = static_cast<float>(acc[k][v]);
                if (tl + k * TS < nq) store_row<VEC>(out + (k < K - 1 ? k * TS * VEC + off : off_last), sum);
            }
        }
        if (next >= more) break;
        run = read_run(table(runs) + next++);
    }
}

// ---- stage 1 for wide rows, every row once, in one pass ------------------------------------------------------------------
// Rows too wide for a workgroup's registers are shared by the workgroups of a *crew*, a contiguous slice of columns each.  Seven
// wavefronts of a member form its parts of the dot products and, a step later, add up the rows; the eighth publishes the member's part
// of every dot product in a slot of its own, one 8-byte word of value and tag, collects the others' and hands out the residuals.  It
// has no rows of its own to wait for, so the exchange (about 1 us) passes behind the loads and the arithmetic of the other seven.
// The members of a crew are 8 workgroup ids apart: on one die where workgroups are dealt to the dies in turn, which is worth a shorter
// exchange and nothing else.  No member depends on another one running: what has not arrived after `patience` polls a member's eighth
// wavefront works out itself, from the rest of the row, in the same order (the same bits), and puts it in the other's slot, where the rest
// of the crew finds it: each member begins with another row.  It waits again once a step's answers are all there at first sight.  Slots are kept
// for all steps, so that a member that starts when the others are done finds their answers.  With 1, 8 or 32 compute units held by another
// stream 4 000 x 50 008 bf16 takes 127 to 134 us with sums (600 to 1 006 with a slot ring of 16 steps, one load in flight and no waiting after
// the first late answer; 133 to 137 in two passes), 20 000 rows 540 to 548 (1 900 to 4 700; 624 to 628).
// A tag is the launch's number and the step's, so that what a slot held before is never taken for an answer: a launch writes every slot
// that it reads, and its number, kept in state[0], is counted up by the last workgroup to finish (state[1] counts those).
// What bounds it is the read of X, 6.5 TB/s over long parts (20 000 x 50 008 bf16, 2 GB, 301 us), and some 10 us to fill the chip and put
// the partial rows away: 4 000 x 50 008 bf16 (400 MB) 75 us against 138 in two passes, 4 000 x 60 000 fp32 (960 MB) 168 against 281.
// What it took: the exchange in a wavefront of its own (loads return in order, so that polls behind a wavefront's own rows wait for
// those: 113 us), two steps for it instead of one (100), rows per step times chunks per thread near eight (two rows instead of four 88),
// no re-reading of the last row at the part's end (82).  Twice the wavefronts with half the chunks each: 107.
template <int XD, int VEC, int K, int R, bool NT>
__global__ void __launch_bounds__(kCrewThreads + 64)
rows_once_crew_kernel(const void *__restrict__ X, const float *__restrict__ y, const float *__restrict__ w, const DevRun *__restrict__ parts,
                      const DevRun *__restrict__ runs, const int32_t *__restrict__ dst, float *__restrict__ rows, int d, int nq, int logistic,
                      int num_parts, int members, uint64_t *slots, int ring_steps, uint32_t *state, int patience)
{
    using C = Chunk<XD, VEC>;
    constexpr int TS = kCrewThreads, WAVES = TS / 64, SETS = 4, LAG = 2;
    static_assert(kCrewMembers * R <= 64, "a lane per slot of a step");
    __shared__ float red[2][R][kCrewThreads / 64], res_of[2][R];
    const int crew = static_cast<int>(blockIdx.x >> 3) / members * 8 + static_cast<int>(blockIdx.x & 7), member = static_cast<int>(blockIdx.x >> 3) % members;
    if (crew >= num_parts) return;
    const int tl = threadIdx.x, lane = tl & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const table_t<DevRun> part = table(parts) + crew;
    const int more = part->more_end;
    int next = part->more_begin;
    Run run = read_run(part);
    const int64_t part_begin = run.row_begin;
    const Run last = next < more ? read_run(table(runs) + (more - 1)) : run;
    const int total = static_cast<int>(last.row_begin + last.nrows - part_begin), steps = (total + R - 1) / R;      // rows past the last one re-read it and count for nothing
    auto slice = [&](int j) { return static_cast<int>(static_cast<int64_t>(nq) * j / members); };       // the last slice is never shorter than another
    // What of chunk q a slice that ends at `end` counts, as bits to keep: an infinity that another lane counts is not to be met by a weight of zero.
    using bits_t = uint32_t __attribute__((ext_vector_type(4)));
    auto owned = [&](int q, int end) {
        bits_t keep = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int v = 0; v < VEC; ++v)
            if (q < end && chunk_owns<VEC>(q, v, nq, d)) keep[v * 4 / VEC] |= VEC == 4 ? ~0u : 0xffffu << v % 2 * 16;
        return keep;
    };
    auto only = [](const typename C::raw_t &x, const bits_t &keep) { return __builtin_bit_cast(typename C::raw_t, __builtin_bit_cast(bits_t, x) & keep); };

    if (wave == WAVES) {
        const uint32_t launch = __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint64_t *const ring = slots + static_cast<int64_t>(crew) * ring_steps * members * R;
        auto targets = [&](int row) { return y[part_begin + min(row + lane, total - 1)]; };
        float y_now = targets(0), y_ahead = targets(64); // of 64 rows each: a load per step would be waited for with the polls
        int y_row = 0;
        // member j's part of the dot product of a row, as its wavefronts form it; as many chunks in flight as there are registers for
        auto part_of_row = [&](int r, int j) {
            constexpr int N = WAVES * K, U = K > 2 ? (N + 1) / 2 : N;
            const int from_q = slice(j), to_q = slice(j + 1);
            const void *row = row_ptr<XD>(X, part_begin + min(r, total - 1), d);
            float p = 0.f, t[2] = {0.f, 0.f};
            auto at = [&](int n) { return from_q + n / K * 64 + lane + n % K * TS; };
#pragma unroll
            for (int n0 = 0; n0 < N; n0 += U) {
                typename C::raw_t x[U];
                float wt[U][VEC];
#pragma unroll
                for (int u = 0; u < U && n0 + u < N; ++u) {
                    const int k = (n0 + u) % K, e = k < K - 1 ? at(n0 + u) * VEC : chunk_offset<VEC>(min(at(n0 + u), to_q - 1), nq, d);
                    x[u] = C::load(row, e);
                    load_row<VEC>(w + e, wt[u]);
                }
#pragma unroll
                for (int u = 0; u < U && n0 + u < N; ++u) {
                    const int q = at(n0 + u), k = (n0 + u) % K;
                    float xv[VEC];
                    C::widen(k < K - 1 ? x[u] : only(x[u], owned(q, to_q)), xv);
#pragma unroll
                    for (int v = 0; v < VEC; ++v)
                        t[k & 1] = fmaf(xv[v], k < K - 1 || (q < to_q && chunk_owns<VEC>(q, v, nq, d)) ? wt[u][v] : 0.f, t[k & 1]);
                    if (k < K - 1) continue;
                    p += group_sum<64>(t[0] + t[1]);
                    t[0] = t[1] = 0.f;
                }
            }
            return p;
        };
        int polls = patience;                            // left for what is late
        for (int i = 0; i < steps + LAG; ++i) {
            auto tag = [&](int step) { return launch << 20 | (static_cast<uint32_t>(step) & 0xfffffu); };
            auto slot = [&](int step) { return ring + (step & (ring_steps - 1)) * members * R; };
            __syncthreads();                             // the wavefronts' parts of step i are in red
            if (i < steps && lane < R) {
                float p = 0.f;
#pragma unroll
                for (int j = 0; j < WAVES; ++j) p += red[i & 1][lane][j];
                __hip_atomic_store(slot(i) + member * R + lane, static_cast<uint64_t>(tag(i)) << 32 | __float_as_uint(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            const int step = i - (LAG - 1);
            if (step < 0 || step >= steps) continue;
            uint64_t word = 0;
            bool here = lane >= members * R;
            auto look = [&] {                            // which slots are still empty
                if (!here) word = __hip_atomic_load(slot(step) + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                here = here || static_cast<uint32_t>(word >> 32) == tag(step);
                return __ballot(!here);
            };
            uint64_t late = look();
            if (!late) polls = patience;
            for (; late && polls > 0; --polls) late = look();
            for (; late; late = look()) {                // what another member has worked out meanwhile is in its slot
                uint64_t choice = late;
                for (int skip = member % __builtin_popcountll(late); skip > 0; --skip) choice &= choice - 1;
                const int at = __builtin_ctzll(choice);
                const float p = part_of_row(step * R + at % R, at / R);
                if (lane == at) {
                    word = static_cast<uint64_t>(tag(step)) << 32 | __float_as_uint(p);
                    here = true;
                    __hip_atomic_store(slot(step) + at, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            const float part_of = __uint_as_float(static_cast<uint32_t>(word));
            float z = 0.f;
            for (int j = 0; j < members; ++j) z += __shfl(part_of, j * R + (lane < R ? lane : 0), 64);
            const int at = step * R + (lane < R ? lane : 0) - y_row;
            const float y0 = __shfl(y_now, at & 63, 64), y1 = __shfl(y_ahead, at & 63, 64);
            if (lane < R) res_of[step & 1][lane] = residual(z, at < 64 ? y0 : y1, logistic);
            if ((step + 1) * R - y_row >= 64) {
                y_row += 64;
                y_now = y_ahead;
                y_ahead = targets(y_row + 64);
            }
        }
        if (lane == 0 && __hip_atomic_fetch_add(state + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == static_cast<uint32_t>(num_parts * members - 1)) {
            __hip_atomic_store(state + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(state, launch + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        return;
    }

    // only a thread's last chunk can be the row's last one or past the slice
    constexpr unsigned kElem = XD == 1 ? 2 : 4;
    const int q_begin = slice(member), q_end = slice(member + 1);
    unsigned off = (q_begin + tl) * VEC, off_last = chunk_offset<VEC>(min(q_begin + tl + (K - 1) * TS, q_end - 1), nq, d);
    float wv[K][VEC];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = q_begin + tl + k * TS;
        load_row<VEC>(w + (k < K - 1 ? k * TS * VEC + off : off_last), wv[k]);
#pragma unroll
        for (int v = 0; v < VEC; ++v) wv[k][v] = q < q_end && chunk_owns<VEC>(q, v, nq, d) ? wv[k][v] : 0.f;
    }
    const int q_last = q_begin + tl + (K - 1) * TS;
    const bool whole = __all(q_last < q_end && (q_last < nq - 1 || d % VEC == 0));
    using Set = typename C::raw_t[R][K];
    Set s[SETS];
    double acc[K][VEC];
    auto clear = [&] {
#pragma unroll
        for (int k = 0; k < K; ++k)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[k][v] = 0.0;
    };
    auto load = [&](Set &x, int step) {
        // the offsets stay 32 bits beside a scalar base: extended once, outside the loop, they would take twice the registers (80 001 bf16 columns 131 against 126 us)
        asm volatile("" : "+v"(off), "+v"(off_last));
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const void *row = row_ptr<XD>(X, part_begin + min(step * R + r, total - 1), d);
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const void *from = static_cast<const char *>(row) + (k < K - 1 ? k * TS * VEC * kElem : 0u);
                const unsigned e = k < K - 1 ? off : off_last;
                x[r][k] = NT ? C::load_once(from, e) : C::load(from, e);
            }
        }
    };
    auto dot = [&](const typename C::raw_t (&x)[K], auto last) {
        float t[2] = {0.f, 0.f};
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float xv[VEC];
            C::widen(k < K - 1 ? x[k] : last(x[k]), xv);
#pragma unroll
            for (int v = 0; v < VEC; ++v) t[k & 1] = fmaf(xv[v], wv[k][v], t[k & 1]);
        }
        return group_sum<64>(t[0] + t[1]);
    };
    auto dots = [&](const Set &x, int step) {
        float p[R], finite = 0.f;
#pragma unroll
        for (int r = 0; r < R; ++r) p[r] = dot(x[r], [](const typename C::raw_t &c) { return c; });
#pragma unroll
        for (int r = 0; r < R; ++r) finite = fmaf(p[r], 0.f, finite);
        // Lanes that count nothing of their last chunk, or not all of it, have weights of zero there, and infinity times zero is no number: once
        // more without.  Four rows at a time: 4 000 x 50 008 bf16 with sums 77.3 us; looked at after every row 82.5, bits masked on every row 78.6.
        if (__builtin_expect(!whole && finite != 0.f, 0)) {
            unsigned at = off;
            asm volatile("" : "+v"(at));                 // worked out here: there are no registers to keep it from step to step
            const bits_t keep = owned(static_cast<int>(at / VEC) + (K - 1) * TS, q_end);
#pragma unroll
            for (int r = 0; r < R; ++r) p[r] = dot(x[r], [&](const typename C::raw_t &c) { return only(c, keep); });
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (lane == 0) red[step & 1][r][wave] = p[r];
    };
    int run_end = run.nrows;                             // rows are counted from the part's first
    auto put_away = [&] {
        for (int j = run.dst_begin; j < run.dst_end; ++j) {
            float *out = rows + static_cast<int64_t>(table(dst)[j]) * d;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                float sum[VEC];
#pragma unroll
                for (int v = 0; v < VEC; ++v) sum[v] = static_cast<float>(acc[k][v]);
                if (q_begin + tl + k * TS < q_end) store_row<VEC>(out + (k < K - 1 ? k * TS * VEC + off : off_last), sum);
            }
        }
        clear();
        if (next >= more) return;
        run = read_run(table(runs) + next++);
        run_end += run.nrows;
    };
    // a chunk to be widened where it is used: the compiler would keep what the dot product widened, or widen ahead of a branch, and there
    // are no registers for that
    auto again = [](typename C::raw_t x) {
        if constexpr (XD == 1) asm volatile("" : "+v"(x));
        return x;
    };
    auto add = [&](const Set &x, int step) {
        const int r0 = step * R;
        float res[R];
#pragma unroll
        for (int r = 0; r < R; ++r) res[r] = res_of[step & 1][r];
        // where a run ends inside a step of several rows: row by row, since a row must not touch another run's sums, not even times zero
        if (R == 1 || r0 + R <= run_end) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                float xv[R][VEC];
#pragma unroll
                for (int r = 0; r < R; ++r) C::widen(again(x[r][k]), xv[r]);
                add_rows<VEC, R>(acc[k], res, xv);
            }
            if (r0 + R == run_end) put_away();
            return;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r0 + r >= total) break;
            const float one[1] = {res[r]};
#pragma unroll
            for (int k = 0; k < K; ++k) {
                float xv[1][VEC];
                C::widen(again(x[r][k]), xv[0]);
                add_rows<VEC, 1>(acc[k], one, xv);
            }
            if (r0 + r + 1 == run_end) put_away();
        }
    };

    clear();
#pragma unroll
    for (int i = 0; i < SETS; ++i) load(s[i], i);
#pragma unroll
    for (int i = 0; i < LAG; ++i) {
        if (i < steps) dots(s[i], i);
        __syncthreads();
    }
    // the dot products of LAG steps are with the eighth wavefront
    int step = 0;
    for (; step + 2 * SETS <= steps; step += SETS) {     // nothing conditional: a load that may not have been issued would be waited for at once
#pragma unroll
        for (int i = 0; i < SETS; ++i) {
            dots(s[(i + LAG) % SETS], step + i + LAG);
            __syncthreads();
            add(s[i], step + i);
            load(s[i], step + i + SETS);
        }
    }
    while (step < steps) {
#pragma unroll
        for (int i = 0; i < SETS; ++i) {
            if (step + LAG < steps) dots(s[(i + LAG) % SETS], step + LAG);
            __syncthreads();
            add(s[i], step);
            if (++step == steps) break;
            if (step + SETS - 1 < steps) load(s[i], step + SETS - 1);
        }
    }
}

// ---- stage 1 for wide rows, every row once ---------------------------------------------------------------------------
// Rows too wide even for a crew, and wide rows of small matrices, whose partial rows would cost more, are read twice: first the residuals phi(x.w) - y of every row
// (R rows per workgroup, so that the weights, twice the size of a bf16 row, come out of the L2 once for R rows), then X^T r by
// blocks of columns and parts of rows.  Both passes are bound by the read of X.  The rows from cached_from on are read with plain
// loads and stay in the last-level cache for the second pass, which takes the parts from the end; the rest streams past (NT).
// 4000 x 50008 bf16 (400 MB) on a (2,4) tree with s = 1: both 124 us; every holder's rows read for itself, in cells of 16 rows, took 1683 us.
template <int XD, int VEC, int R>
__global__ void __launch_bounds__(512)
wide_residuals_kernel(const void *__restrict__ X, const float *__restrict__ y, const float *__restrict__ w, float *__restrict__ residuals,
                      int64_t m, int d, int nq, int logistic, int64_t cached_from)
{
    using C = Chunk<XD, VEC>;
    constexpr int U = 8 / R, WAVES = 8;                  // eight row chunks in flight per thread
    const int64_t r0 = static_cast<int64_t>(blockIdx.x) * R;
    float s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = 0.f;
    auto pass = [&](auto nt) {
        for (int b = 0; b < nq; b += 512 * U) {
            typename C::raw_t x[U][R];
            float wv[U][VEC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int off = chunk_offset<VEC>(b + u * 512 + static_cast<int>(threadIdx.x), nq, d);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const void *row = row_ptr<XD>(X, min(r0 + r, m - 1), d);
                    x[u][r] = decltype(nt)::value ? C::load_once(row, off) : C::load(row, off);
                }
                load_row<VEC>(w + off, wv[u]);
            }
            const bool whole = b + 512 * U < nq;         // no thread's chunk is the row's last one, which may overlap its neighbour
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    float xv[VEC];
                    C::widen(x[u][r], xv);
                    if (whole) {
#pragma unroll
                        for (int v = 0; v < VEC; ++v) s[r] = fmaf(xv[v], wv[u][v], s[r]);
                    } else {
                        const int q = b + u * 512 + static_cast<int>(threadIdx.x);
#pragma unroll
                        for (int v = 0; v < VEC; ++v)
                            if (chunk_owns<VEC>(q, v, nq, d)) s[r] = fmaf(xv[v], wv[u][v], s[r]);
                    }
                }
        }
    };
    if (r0 >= cached_from) pass(std::false_type{});
    else pass(std::true_type{});
    __shared__ float red[R][WAVES];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float t = group_sum<64>(s[r]);
        if ((threadIdx.x & 63) == 0) red[r][threadIdx.x >> 6] = t;
    }
    __syncthreads();
    const int r = threadIdx.x;
    if (r >= R || r0 + r >= m) return;
    float z = 0.f;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) z += red[r][i];
    residuals[r0 + r] = residual(z, y[r0 + r], logistic);
}

template <int XD, int VEC>
__global__ void __launch_bounds__(256)
wide_xt_kernel(const void *__restrict__ X, const float *__restrict__ residuals, const DevRun *__restrict__ parts, const DevRun *__restrict__ runs,
               const int32_t *__restrict__ dst, float *__restrict__ rows, int d, int nq, int64_t cached_from)
{
    using C = Chunk<XD, VEC>;
    constexpr int U = 16;                                // rows in flight
    const table_t<DevRun> part = table(parts) + (gridDim.y - 1 - blockIdx.y);
    const int more = part->more_end;
    int next = part->more_begin;
    Run run = read_run(part);
    const int q = blockIdx.x * 256 + threadIdx.x;        // threads past the row repeat its last chunk and do not store
    const int off = chunk_offset<VEC>(q, nq, d);
    const bool cached = run.row_begin >= cached_from;
    for (;;) {
        const void *base = row_ptr<XD>(X, run.row_begin, d);
        const float *res = residuals + run.row_begin;
        const int n = run.nrows;
        double acc[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
        auto pass = [&](auto nt) {
            for (int r0 = 0; r0 < n; r0 += U) {
                typename C::raw_t x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const void *row = row_ptr<XD>(base, min(r0 + u, n - 1), d);
                    x[u] = decltype(nt)::value ? C::load_once(row, off) : C::load(row, off);
                }
#pragma unroll
                for (int u = 0; u < U; u += 4) {
                    float xv[4][VEC], rv[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        C::widen(x[u + i], xv[i]);
                        rv[i] = r0 + u + i < n ? res[r0 + u + i] : 0.f;
                    }
                    add_rows<VEC, 4>(acc, rv, xv);
                }
            }
        };
        if (cached) pass(std::false_type{});
        else pass(std::true_type{});
        float sum[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) sum[v] = static_cast<float>(acc[v]);
        if (q < nq)
            for (int j = run.dst_begin; j < run.dst_end; ++j) store_row<VEC>(rows + static_cast<int64_t>(table(dst)[j]) * d + off, sum);
        if (next >= more) break;
        run = read_run(table(runs) + next++);
    }
}

// ---- stage 1 for wide rows, every holder separately ----------------------------------------------------------------
// When a row is too long for one team's registers the single pass is split in two: first the residuals r = phi(x.w) - y of every
// row visit (one workgroup per piece, the row streamed in chunks), then G_piece = X^T r per piece and column block.
template <int XD, int VEC>
__global__ void __launch_bounds__(256)
residuals_kernel(const void *__restrict__ X, const float *__restrict__ y, const float *__restrict__ w,
                 const DevPiece *__restrict__ pieces, float *__restrict__ residuals, int d, int nq, int logistic)
{
    using C = Chunk<XD, VEC>;
    using raw_t = typename C::raw_t;
    constexpr int U = 8;                                 // chunks in flight per thread
    const DevPiece pc = pieces[blockIdx.x];
    __shared__ float red[2][4];
    int buf = 0;
    for (int r = 0; r < pc.nrows; ++r) {
        const void *row = row_ptr<XD>(X, pc.row_begin + r, d);
        float s = 0.f;
        for (int q0 = threadIdx.x; q0 < nq; q0 += 256 * U) {
            raw_t xr[U];
#pragma unroll
            for (int u = 0; u < U; ++u) xr[u] = C::load(row, chunk_offset<VEC>(q0 + u * 256, nq, d));
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int q = q0 + u * 256;
                const int o = chunk_offset<VEC>(q, nq, d);
                float xv[VEC];
                C::widen(xr[u], xv);
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                    if (chunk_owns<VEC>(q, v, nq, d)) s = fmaf(xv[v], w[o + v], s);
            }
        }
        s = wave_sum<true>(s);
        if ((threadIdx.x & 63) == 0) red[buf][threadIdx.x / 64] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            const float z = red[buf][0] + red[buf][1] + red[buf][2] + red[buf][3];
            const float ph = logistic ? sigmoid(z) : z;
            residuals[pc.visit_begin + r] = ph - y[pc.row_begin + r];
        }
        buf ^= 1;
    }
}

template <int XD, int VEC>
__global__ void __launch_bounds__(256)
xt_residuals_kernel(const void *__restrict__ X, const DevPiece *__restrict__ pieces, const float *__restrict__ residuals,
                    float *__restrict__ rows, int d, int nq)
{
    using C = Chunk<XD, VEC>;
    using raw_t = typename C::raw_t;
    constexpr int K = kWideChunks;
    const DevPiece pc = pieces[blockIdx.y];
    const int qbase = blockIdx.x * (256 * K) + threadIdx.x;
    unsigned off[K];
#pragma unroll
    for (int k = 0; k < K; ++k) off[k] = chunk_offset<VEC>(qbase + k * 256, nq, d);
    float acc[K][VEC];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[k][v] = 0.f;
    for (int r = 0; r < pc.nrows; ++r) {
        const void *row = row_ptr<XD>(X, pc.row_begin + r, d);
        const float res = residuals[pc.visit_begin + r];
        raw_t xr[K];
#pragma unroll
        for (int k = 0; k < K; ++k) xr[k] = C::load(row, off[k]);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float xv[VEC];
            C::widen(xr[k], xv);
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[k][v] = fmaf(res, xv[v], acc[k][v]);
        }
    }
    float *out = rows + static_cast<int64_t>(pc.out_row) * d;
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (qbase + k * 256 < nq) store_row<VEC>(out + off[k], acc[k]);
}

// ---- sums of partial rows ---------------------------------------------------------------------------------------------
// Slabs that several runs make up: the sum of consecutive partial rows, written to every slab that covers the same rows (so the
// partial rows are read once per distinct slab range, not once per slab).  A workgroup covers 64 chunks of columns of one sum; its
// eight wavefronts each add every eighth row (eight loads in flight per lane), the eight partial sums meet in LDS, and the
// wavefronts share out the destinations.  fp64 throughout, in an order fixed by the tables alone: the same bits on every run.
template <int VEC>
__global__ void __launch_bounds__(512)
sum_rows_kernel(float *__restrict__ rows, const DevSum *__restrict__ sums, const int32_t *__restrict__ dst, int64_t d, int nq)
{
    constexpr int WAVES = 8, U = 8;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = min(static_cast<int>(blockIdx.x) * 64 + lane, nq - 1);     // lanes past the row repeat its last chunk and do not store
    const int64_t col = chunk_offset<VEC>(q, nq, static_cast<int>(d));
    const table_t<DevSum> s = table(sums) + blockIdx.y;
    const int row_begin = s->row_begin, row_end = s->row_end;
    double acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
    for (int j0 = row_begin + wave; j0 < row_end; j0 += WAVES * U) {
        float xv[U][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) load_row<VEC>(rows + static_cast<int64_t>(min(j0 + u * WAVES, row_end - 1)) * d + col, xv[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j0 + u * WAVES < row_end) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] += static_cast<double>(xv[u][v]);
            }
    }
    __shared__ double part[WAVES][VEC][64];
#pragma unroll
    for (int v = 0; v < VEC; ++v) part[wave][v][lane] = acc[v];
    __syncthreads();
    if (static_cast<int>(blockIdx.x) * 64 + lane >= nq) return;
    float out[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < WAVES; ++i) t += part[i][v][lane];
        out[v] = static_cast<float>(t);
    }
    for (int j = s->dst_begin + wave; j < s->dst_end; j += WAVES) store_row<VEC>(rows + static_cast<int64_t>(table(dst)[j]) * d + col, out);
}

// The same for many sums of few rows (see launch_sum_rows): a wavefront per 64 chunks of columns takes all rows of a sum, in their order, where
// the workgroup above would have wavefronts without a row and eight times the workgroups.
__global__ void __launch_bounds__(256)
sum_few_rows_kernel(float *__restrict__ rows, const DevSum *__restrict__ sums, const int32_t *__restrict__ dst, int64_t d, int nq)
{
    constexpr int VEC = 4, U = 8;
    const int q = blockIdx.x * 256 + threadIdx.x;
    const int64_t col = chunk_offset<VEC>(min(q, nq - 1), nq, static_cast<int>(d));
    const table_t<DevSum> s = table(sums) + blockIdx.y;
    const int row_begin = s->row_begin, row_end = s->row_end, dst_begin = s->dst_begin, dst_end = s->dst_end;
    double acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
    for (int j0 = row_begin; j0 < row_end; j0 += U) {
        float xv[U][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) load_row<VEC>(rows + static_cast<int64_t>(min(j0 + u, row_end - 1)) * d + col, xv[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j0 + u < row_end) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] += static_cast<double>(xv[u][v]);
            }
    }
    if (q >= nq) return;
    float out[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) out[v] = static_cast<float>(acc[v]);
    for (int j = dst_begin; j < dst_end; ++j) store_row<VEC>(rows + static_cast<int64_t>(table(dst)[j]) * d + col, out);
}

// ---- encode ---------------------------------------------------------------------------------------------------------
// One thread owns C chunks of VEC columns and runs the whole sub-tree of one level-1 node for them: a post-order list of terms
// (own += coef * G[slab]) in which the last term of a node finishes it: message = own + pending[level], stored (rounded to fp32,
// as a transmitted message would be) and folded into pending[level-1] with the parent's decode coefficient.  Child messages
// therefore never come back from HBM; every active slab is read once and every message written once.  The program is the same for
// every thread, so it is read with wide scalar loads, U terms at a time; the slab loads of those terms are all issued before the
// first is used.  Slabs are touched once: non-temporal loads.  Messages of short vectors are written the ordinary way, since the decode
// reads some of them and the next mask's replace them; those of long ones are non-temporal too (3 000 000 columns: 509 against 557 us).
// A workgroup of BS threads covers BS*C*VEC contiguous columns of every row it touches.  Two shapes are used:
//   narrow  C=1, U=8, fp64 accumulators: for short vectors, where the launch has few threads and latency decides;
//   wide    C=32, U=1, fp32 accumulators: for long vectors.  A workgroup then streams 128 KB-aligned, 128 KB-long pieces of one
//           slab at a time, which is what HBM likes best (the same 31-stream pattern read 4 KB at a time reaches 4.9 TB/s, this
//           6.1 TB/s); the 32 chunks in flight fill the register file, hence fp32 accumulation: two or three extra roundings
//           of the size of the message's own fp32 rounding.
// walk_sub_tree: terms [tb, te) of a program for a thread's C chunks, off bytes into a row; live: is the chunk in the row; top(c, out): the
// finished message of the level-1 node.
template <int VEC, int LT, int C, int U, bool NTS, typename acc_t, typename TOP>
__device__ __forceinline__ void walk_sub_tree(const float *G, float *M, const EncProgram &prog, int tb, int te, int64_t d, const unsigned (&off)[C],
                                              const bool (&live)[C], TOP top)
{
    static_assert(kEncodeUnroll % U == 0, "sub-programs are padded to kEncodeUnroll terms");
    typedef int iuv __attribute__((ext_vector_type(U)));
    typedef double duv __attribute__((ext_vector_type(U)));
    acc_t pend[LT + 1][C][VEC];
    acc_t own[C][VEC];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            own[c][v] = 0;
#pragma unroll
            for (int l = 0; l <= LT; ++l) pend[l][c][v] = 0;
        }

    for (int t = tb; t < te; t += U) {
        const iuv slab = *table(reinterpret_cast<const iuv *>(prog.slab + t));
        const iuv level = *table(reinterpret_cast<const iuv *>(prog.level + t));
        const iuv row = *table(reinterpret_cast<const iuv *>(prog.row + t));
        const duv coef = *table(reinterpret_cast<const duv *>(prog.coef + t));
        const duv acoef = *table(reinterpret_cast<const duv *>(prog.acoef + t));
        float xv[U][C][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float *src = G + static_cast<int64_t>(slab[u]) * d;      // the same for all lanes: a scalar base and the lane's 32-bit offset
#pragma unroll
            for (int c = 0; c < C; ++c) load_row_nt<VEC>(at_byte(src, off[c]), xv[u][c]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int c = 0; c < C; ++c)
#pragma unroll
                for (int v = 0; v < VEC; ++v) own[c][v] = fma(static_cast<acc_t>(coef[u]), static_cast<acc_t>(xv[u][c][v]), own[c][v]);
            const int lvl = level[u];
            if (lvl > 0) {
                float *dst = M + static_cast<int64_t>(row[u]) * d;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    float out[VEC];
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        acc_t msg = own[c][v];
#pragma unroll
                        for (int l = 1; l < LT; ++l)               // only levels 1..L-1 ever collect children
                            if (l == lvl) { msg += pend[l][c][v]; pend[l][c][v] = 0; }
                        out[v] = static_cast<float>(msg);
                        own[c][v] = 0;
                    }
                    if (live[c] && row[u] >= 0) {
                        if constexpr (NTS) store_row_nt<VEC>(at_byte(dst, off[c]), out);
                        else store_row<VEC>(at_byte(dst, off[c]), out);
                    }
                    if (lvl == 1) top(c, out);
#pragma unroll
                    for (int l = 1; l < LT; ++l)
                        if (l == lvl - 1) {
#pragma unroll
                            for (int v = 0; v < VEC; ++v) pend[l][c][v] = fma(static_cast<acc_t>(acoef[u]), static_cast<acc_t>(out[v]), pend[l][c][v]);
                        }
                }
            }
        }
    }
}

template <int VEC, int LT, int C, int BS, int U, bool NTS, typename acc_t>
__global__ void __launch_bounds__(BS)
encode_kernel(const float *__restrict__ G, float *__restrict__ M, EncProgram prog, int64_t d, int nq)
{
    const int q0 = blockIdx.x * (BS * C) + threadIdx.x;
    if (q0 >= nq) return;
    // whole groups of U terms: the padding terms are only fetched when U does not divide the real length
    const int tb = prog.sub_begin[blockIdx.y], te = tb + (prog.sub_end[blockIdx.y] - tb + U - 1) / U * U;
    // chunk c of this thread; a chunk past the end of the row is redirected to the row's last chunk and not stored
    unsigned off[C];
    bool live[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int q = q0 + c * BS;
        live[c] = q < nq;
        off[c] = 4u * chunk_offset<VEC>(q, nq, static_cast<int>(d));
    }
    walk_sub_tree<VEC, LT, C, U, NTS, acc_t>(G, M, prog, tb, te, d, off, live, [](int, const float (&)[VEC]) {});
}

// Encode and decode of several masks, one after the other, in one launch: a workgroup owns 64 chunks of columns for all of them, its
// wavefronts share out the level-1 sub-trees, whose messages meet in LDS for the decode (two sets in turn: one barrier per mask, after
// which one wavefront decodes while the others go on).  No launches, ramps and last waves between the masks, and the master's messages
// are not read back.  us a mask of eight, a launch each for encode and decode / this: (2,4) tree, 2 000 000 columns 50.9 / 48.1; (3,4), 60 001
// columns 13.6 / 10.7; (2,12), s = 5, 117 706 columns 51.9 / 49.4 (rows on 8-byte boundaries; 117 760 columns 50.6 / 47.7).  Where it loses: see
// encode_in_steps.  Slabs are read past the caches.  Messages that a later mask replaces are not written at all (row < 0): 117 706 columns,
// s = 5, 51 us a mask, 62 with every one written.
template <int LT>
__global__ void __launch_bounds__(1024)
encode_steps_kernel(const float *__restrict__ G, int64_t G_stride, float *__restrict__ M, EncProgram prog, int64_t prog_stride, int steps, int n,
                    float *__restrict__ g, int64_t g_stride, int64_t d, int nq)
{
    constexpr int VEC = 4;
    extern __shared__ __align__(16) char step_lds[];
    float *top = reinterpret_cast<float *>(step_lds);    // [2][n][VEC][64]
    const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // workgroups are dealt to the eight dies in turn: neighbouring columns on one die, whose L2 joins the lines they share (with another
    // number of dies the same columns, on others)
    const int block = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3), q = block * 64 + lane;
    if (block * 64 >= nq) return;
    const bool live[1] = {q < nq};
    const unsigned off[1] = {4u * chunk_offset<VEC>(q, nq, static_cast<int>(d))};
    for (int t = 0; t < steps; ++t) {
        float *set = top + (t & 1) * n * VEC * 64;
        EncProgram p = prog.at(t * prog_stride);
        for (int i = wave; i < n; i += waves) {
            const int tb = table(p.sub_begin)[i], te = tb + (table(p.sub_end)[i] - tb + kEncodeUnroll - 1) / kEncodeUnroll * kEncodeUnroll;
            walk_sub_tree<VEC, LT, 1, kEncodeUnroll, false, double>(G + t * G_stride, M, p, tb, te, d, off, live, [&](int, const float (&out)[VEC]) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) set[(i * VEC + v) * 64 + lane] = out[v];
            });
        }
        __syncthreads();
        if (wave != t % waves) continue;
        double acc[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
        for (int j = 0; j < n; ++j) {
            const double a = table(p.dec)[j];                   // zero: not used
            if (a == 0.0) continue;
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[v] = fma(a, static_cast<double>(set[(j * VEC + v) * 64 + lane]), acc[v]);
        }
        float out[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) out[v] = static_cast<float>(acc[v]);
        if (live[0]) store_row<VEC>(at_byte(g + t * g_stride, off[0]), out);
    }
}

// ---- encode, the nodes of a tree side by side ---------------------------------------------------------------------------
// The encode of short vectors takes as long as its chain of dependent fetches, not its bytes: a thread that walks a whole sub-tree
// fetches eight terms at a time, one group after the other.  Here B lanes own B chunks of columns and the workgroup's T / B teams
// share out the nodes: all form their own sums at once (one fetch of a node's entries, one of its slabs), the messages meet in LDS
// and the levels above the leaves fold their children from there, one barrier per level.  Sums are fp64, formed in the order in which
// encode_kernel forms them, and messages are rounded where it rounds them: the same bits.
// What the mask decides, a coefficient per node, travels as kernel arguments, so there is no copy to wait for; the tree's tables are on
// the device beside the slabs that stage 1 leaves there, or travel as arguments too.
// Kernel time in us, a thread per sub-tree / nodes side by side: (2,12) tree, s = 2, 10 columns 7.5 / 4.2; s = 3, 5 001 columns
// 12.5 / 5.9; (3,6) tree, s = 2, 1 024 columns 25.9 / 6.7; (3,4) tree, 6 500 columns 8.5 / 5.7.
__device__ __forceinline__ bool sends(double a) { return __double_as_longlong(a) != kStraggler; }

// A workgroup's view of the tables: read in place where they are on the device ...
template <typename TABLES> struct DeviceView {
    const TABLES &t;
    __device__ __forceinline__ double coef_of(int node) const { return t.coefs.a[node]; }
    __device__ __forceinline__ int begin(int node) const { return t.node_begin[node]; }
    __device__ __forceinline__ double slab_coef_of(int s) const { return t.slab_coef[s]; }
};
__device__ __forceinline__ DeviceView<DeviceTables> view_tables(const DeviceTables &t, int, char *) { return {t}; }
__device__ __forceinline__ DeviceView<SmallDeviceTables> view_tables(const SmallDeviceTables &t, int, char *) { return {t}; }
// ... and copied to LDS first where they are arguments, since a coefficient is two dependent fetches away.
struct ArgumentView {
    const double *value;
    const uint16_t *first, *coef, *slab;
    __device__ __forceinline__ double coef_of(int node) const { return value[coef[node]]; }
    __device__ __forceinline__ int begin(int node) const { return first[node]; }
    __device__ __forceinline__ double slab_coef_of(int s) const { return value[slab[s]]; }
};
template <typename TABLES> __device__ __forceinline__ ArgumentView view_arguments(const TABLES &t, int threads, char *lds)
{
    uint64_t *copy = reinterpret_cast<uint64_t *>(lds);
    for (int i = threadIdx.x; i < t.used; i += threads) copy[i] = t.word[i];
    __syncthreads();
    const uint16_t *half = reinterpret_cast<const uint16_t *>(lds);
    return {reinterpret_cast<const double *>(lds), half + t.at_begin, half + t.at_coef, half + t.at_slab};
}
__device__ __forceinline__ ArgumentView view_tables(const ArgumentTables &t, int threads, char *lds) { return view_arguments(t, threads, lds); }
__device__ __forceinline__ ArgumentView view_tables(const SmallArgumentTables &t, int threads, char *lds) { return view_arguments(t, threads, lds); }

// The places of a workgroup's nodes, leaves first, then level by level up; sub: which level-1 sub-tree (0 where it has them all).
struct TreePlaces {
    const TreeLevels &tree;
    int sub;
    __device__ __forceinline__ int node(int t) const
    {
        int id = t + tree.shift[tree.L - 1] + sub * tree.width[tree.L - 1];
        for (int l = tree.L - 1; l >= 1; --l)
            if (t >= tree.first[l - 1]) id = t + tree.shift[l - 1] + sub * tree.width[l - 1];
        return id;
    }
};

// LDS of a workgroup that has `total` nodes, `total - leaves` of them above the leaves
template <int VEC, int B> struct TreeLds {
    static __host__ __device__ size_t bytes(int total, int leaves) { return static_cast<size_t>(total) * (B * VEC * 4 + 8) + static_cast<size_t>(total - leaves) * B * VEC * 8; }
    double *coef;                                        // [total]: with which the node's message is folded in
    double *own;                                         // [total - leaves][VEC][B]: own sums of the nodes above the leaves
    float *msg;                                          // [total][VEC][B]: messages
    __device__ __forceinline__ TreeLds(char *at, int total, int leaves)
        : coef(reinterpret_cast<double *>(at)), own(coef + total), msg(reinterpret_cast<float *>(own + (total - leaves) * VEC * B)) {}
    __device__ __forceinline__ void put_message(int t, int tl, const float (&m)[VEC]) const
    {
#pragma unroll
        for (int v = 0; v < VEC; ++v) msg[(t * VEC + v) * B + tl] = m[v];
    }
    // acc += coef * message, the nodes [t0, t0 + n) in turn, four read at a time; SKIP: those with coefficient zero are left out
    template <bool SKIP> __device__ __forceinline__ void fold(int t0, int n, int tl, double (&acc)[VEC]) const
    {
        constexpr int U = 4;
        for (int c0 = 0; c0 < n; c0 += U) {
            double a[U];
            float m[U][VEC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int t = t0 + min(c0 + u, n - 1);
                a[u] = coef[t];
#pragma unroll
                for (int v = 0; v < VEC; ++v) m[u][v] = msg[(t * VEC + v) * B + tl];
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (c0 + u < n && sends(a[u]) && !(SKIP && a[u] == 0.0)) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[v] = fma(a[u], static_cast<double>(m[u][v]), acc[v]);
                }
        }
    }
};

// own sum of a node: its slabs in turn, U of them in flight
template <int VEC, typename COEF>
__device__ __forceinline__ void sum_slabs(const float *G, int64_t d, int64_t col, int begin, int end, COEF coef, double (&acc)[VEC])
{
    constexpr int U = 8;
    for (int s0 = begin; s0 < end; s0 += U) {
        float x[U][VEC];
        double c[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u < end) {
                load_row<VEC>(G + static_cast<int64_t>(s0 + u) * d + col, x[u]);
                c[u] = coef(s0 + u);
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (s0 + u < end) {
#pragma unroll
                for (int v = 0; v < VEC; ++v) acc[v] = fma(c[u], static_cast<double>(x[u][v]), acc[v]);
            }
    }
}

// The messages of a workgroup's nodes, stored and left in LDS.
template <int VEC, int B, typename VIEW>
__device__ __forceinline__ void tree_messages(const TreeLevels &tree, int sub, const TreeLds<VEC, B> &lds, const VIEW &view, const NodeBits &stored,
                                              const float *G, float *M, int64_t d, int64_t col, bool live)
{
    const int TEAMS = tree.threads / B;
    // 64 lanes: the team is a wavefront, and what it reads of the tables is the same for all lanes
    const int team = B == 64 ? __builtin_amdgcn_readfirstlane(threadIdx.x / 64) : threadIdx.x / B, tl = threadIdx.x % B;
    const TreePlaces places{tree, sub};
    auto stores = [&](int node) { return (stored.word[node >> 5] >> (node & 31) & 1u) != 0; };
    for (int t = team; t < tree.total; t += TEAMS) {
        const int node = places.node(t);
        const double a = view.coef_of(node);
        const bool put_down = stores(node);
        const int begin = view.begin(node), end = view.begin(node + 1);
        if (tl == 0) lds.coef[t] = a;
        if (!sends(a)) continue;
        double acc[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
        sum_slabs<VEC>(G, d, col, begin, end, [&](int s) { return view.slab_coef_of(s); }, acc);
        if (t < tree.leaves) {
            float out[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) out[v] = static_cast<float>(acc[v]);
            if (live && put_down) store_row<VEC>(M + static_cast<int64_t>(node) * d + col, out);
            lds.put_message(t, tl, out);
        } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v) lds.own[((t - tree.leaves) * VEC + v) * B + tl] = acc[v];
        }
    }
    for (int l = tree.L - 1; l >= 1; --l) {
        __syncthreads();
        const int first = tree.first[l - 1], end = l > 1 ? tree.first[l - 2] : tree.total;
        for (int t = first + team; t < end; t += TEAMS) {
            if (!sends(lds.coef[t])) continue;
            const int node = places.node(t);
            const bool put_down = stores(node);
            double pend[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) pend[v] = 0.0;
            lds.template fold<false>(tree.first[l] + (t - first) * tree.n, tree.n, tl, pend);
            float out[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) out[v] = static_cast<float>(lds.own[((t - tree.leaves) * VEC + v) * B + tl] + pend[v]);
            if (live && put_down) store_row<VEC>(M + static_cast<int64_t>(node) * d + col, out);
            lds.put_message(t, tl, out);
        }
    }
}

// one level-1 sub-tree (grid.y) per workgroup
template <int VEC, int B, typename TABLES>
__global__ void __launch_bounds__(1024)
tree_kernel(const float *__restrict__ G, float *__restrict__ M, TABLES tables, NodeBits stored, TreeLevels tree, int64_t d, int nq)
{
    extern __shared__ __align__(16) char tree_lds[];
    const auto view = view_tables(tables, tree.threads, tree_lds);
    const TreeLds<VEC, B> lds(tree_lds + TABLES::kLdsBytes, tree.total, tree.leaves);
    const int q = blockIdx.x * B + threadIdx.x % B;
    const int64_t col = chunk_offset<VEC>(q, nq, static_cast<int>(d));       // lanes past the row repeat its last chunk and do not store
    tree_messages<VEC, B>(tree, blockIdx.y, lds, view, stored, G, M, d, col, q < nq);
}

// What one column contributes to the convergence measures of a gradient step: |w_new - w|^2, |w|^2, |w_new - w*|^2, |w*|^2.
__device__ __forceinline__ void measure(double (&sum)[4], float w_old, float w_new, bool with_star, float w_star)
{
    const double dw = static_cast<double>(w_new) - static_cast<double>(w_old);
    sum[0] += dw * dw;
    sum[1] += static_cast<double>(w_old) * w_old;
    if (with_star) {
        const double ws = w_star, e = static_cast<double>(w_new) - ws;
        sum[2] += e * e;
        sum[3] += ws * ws;
    }
}

// What the step reads of the chunk at column col.  The chunk that owns a column is the only one that uses and writes its entry.
template <int VEC> __device__ __forceinline__ void load_step(const GradientStep &step, int64_t col, float (&w_old)[VEC], float (&w_star)[VEC])
{
    if (step.w) load_row<VEC>(step.w + col, w_old);
    if (step.measures && step.w_star) load_row<VEC>(step.w_star + col, w_star);
}

// The decoded chunk q goes to g; step.w: w <- w - lr g with g as stored, a column shared with the neighbouring chunk by the chunk that
// owns it only; step.measures: the columns' part of the measures is added to sum.  SAME: w, g and w_star may be one vector,
// and the values are those of a launch each for decode, step and measures.  (In tree_decode_kernel it cost 20 steps on 1 200 x 100 3 us of 218.)
template <int VEC, bool NT, bool SAME>
__device__ __forceinline__ void put_gradient(const double (&acc)[VEC], float *g, int64_t col, int q, int nq, int64_t d, const GradientStep &step,
                                             const float (&w_old)[VEC], const float (&w_star)[VEC], double (&sum)[4])
{
    float out[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) out[v] = static_cast<float>(acc[v]);
    const bool g_is_w = SAME && step.w == g, star_is_w = SAME && step.w_star == step.w, star_is_g = SAME && step.w_star == g;
    if (!g_is_w) {
        if constexpr (NT) store_row_nt<VEC>(g + col, out);
        else store_row<VEC>(g + col, out);
    }
    if (!step.w) return;
#pragma unroll
    for (int v = 0; v < VEC; ++v)
        if (chunk_owns<VEC>(q, v, nq, static_cast<int>(d))) {
            const float before = g_is_w ? out[v] : w_old[v], w_new = fmaf(-step.lr, out[v], before);
            step.w[col + v] = w_new;
            if (step.measures) measure(sum, before, w_new, step.w_star != nullptr, star_is_w ? w_new : star_is_g ? out[v] : w_star[v]);
        }
}

// The whole tree per workgroup, the master's decode and the gradient step after it: one launch where there were two or three.  For
// vectors of so few columns that a launch lasts no longer than its chain of fetches; longer ones have more to gain from a workgroup per
// sub-tree and a decode of their own.  us of encode and decode, apart / together, 16 masks back to back: (2,4) tree, 1 024 columns 5.7 / 4.3; (2,12),
// s = 2, 10 columns 6.6 / 5.2, 1 024 6.8 / 6.0, 16 384 11.6 / 11.1, 73 728 27.8 / 38.1; (3,4), 6 500 columns 8.3 / 6.3, 32 768 10.3 / 9.7.
template <int VEC, int B, typename TABLES>
__global__ void __launch_bounds__(1024)
tree_decode_kernel(const float *__restrict__ G, float *__restrict__ M, TABLES tables, NodeBits stored, TreeLevels tree, float *__restrict__ g,
                   GradientStep step, int64_t d, int nq)
{
    extern __shared__ __align__(16) char tree_lds[];
    const auto view = view_tables(tables, tree.threads, tree_lds);
    const TreeLds<VEC, B> lds(tree_lds + TABLES::kLdsBytes, tree.total, tree.leaves);
    const int tl = threadIdx.x % B, q = blockIdx.x * B + tl;
    const int64_t col = chunk_offset<VEC>(q, nq, static_cast<int>(d));
    float w_old[VEC] = {}, w_star[VEC] = {};             // on their way from the start, not once the gradient is there
    if (threadIdx.x < B) load_step<VEC>(step, col, w_old, w_star);
    tree_messages<VEC, B>(tree, 0, lds, view, stored, G, M, d, col, q < nq);
    __syncthreads();
    if (threadIdx.x >= B) return;
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    if (q < nq) {
        double acc[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = 0.0;
        lds.template fold<true>(tree.first[0], tree.n, tl, acc);
        put_gradient<VEC, false, false>(acc, g, col, q, nq, d, step, w_old, w_star, sum);
    }
    if (!step.measures) return;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int o = B / 2; o > 0; o >>= 1) sum[k] += __shfl_xor(sum[k], o, 64);
        if (tl == 0) step.measures[4 * blockIdx.x + k] = sum[k];
    }
}

// ---- decode ---------------------------------------------------------------------------------------------------------
// The terms come as kernel arguments.  A thread owns C chunks of columns, 256 chunks apart, and has U rows of them in flight: eight rows
// of one chunk where latency decides, one row of four chunks, past the caches, for long vectors, where HBM prefers long pieces of one
// row (six rows of 16 777 216 columns: 92 us with eight rows of one chunk, 83 one by one, 79 in this shape; 4 000 000: 23.4, 23.2, 22.3;
// 1 000 000: 8.7, 8.6, 8.5; two rows of 2 500 000: 8.8 one by one, 8.4 in this shape, of 1 634 474, where its 400 workgroups fill the chip one
// and a half times: 7.4, 8.1).
constexpr int64_t kDecodeLongColumns = int64_t(1) << 21;
template <int VEC, int U, int C, bool NT>
__global__ void __launch_bounds__(256)
decode_kernel(const float *__restrict__ M, float *__restrict__ g, DecTerms terms, GradientStep step, int64_t d, int nq)
{
    const int q0 = blockIdx.x * (256 * C) + threadIdx.x;
    int64_t col[C];                                      // chunks past the row repeat its last one and are not stored
    double acc[C][VEC];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        col[c] = chunk_offset<VEC>(q0 + c * 256, nq, static_cast<int>(d));
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[c][v] = 0.0;
    }
    for (int j0 = 0; j0 < terms.count; j0 += U) {
        float xv[U][C][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j0 + u < terms.count) {
                const float *src = M + static_cast<int64_t>(terms.row[j0 + u]) * d;
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    if constexpr (NT) load_row_nt<VEC>(src + col[c], xv[u][c]);
                    else load_row<VEC>(src + col[c], xv[u][c]);
                }
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j0 + u < terms.count) {
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[c][v] = fma(terms.coef[j0 + u], static_cast<double>(xv[u][c][v]), acc[c][v]);
            }
    }
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < C; ++c) {
        float w_old[VEC] = {}, w_star[VEC] = {};
        load_step<VEC>(step, col[c], w_old, w_star);
        if (q0 + c * 256 < nq) put_gradient<VEC, NT, true>(acc[c], g, col[c], q0 + c * 256, nq, d, step, w_old, w_star, sum);
    }
    if (!step.measures) return;
    __shared__ double part[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum[k] += __shfl_xor(sum[k], o, 64);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][k] = sum[k];
    }
    __syncthreads();
    if (threadIdx.x < 4) step.measures[4 * blockIdx.x + threadIdx.x] = part[0][threadIdx.x] + part[1][threadIdx.x] + part[2][threadIdx.x] + part[3][threadIdx.x];
}

__global__ void __launch_bounds__(256) update_kernel(float *__restrict__ w, const float *__restrict__ g, float lr, int64_t d)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < d) w[i] = fmaf(-lr, g[i], w[i]);
}

// The two convergence measures of the paper's experiments, one workgroup per step, from what the launches that made the steps left, four
// sums per workgroup: metrics[0] = ||w_new - w||^2 / ||w||^2 (relative error rate, eq. (6)), metrics[1] = ||w_new - w*||^2 / ||w*||^2
// (normalised error rate, eq. (8)), or -1 without w*.  Fixed summation order.
__global__ void __launch_bounds__(256)
measures_kernel(const double *__restrict__ sums, int64_t step_stride, int groups, bool with_star, float *__restrict__ metrics)
{
    const double *s = sums + blockIdx.x * step_stride;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < groups; i += 256)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] += s[4 * static_cast<int64_t>(i) + k];
    __shared__ double part[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) acc[k] += __shfl_xor(acc[k], o, 64);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][k] = acc[k];
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double tot[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) tot[k] = part[0][k] + part[1][k] + part[2][k] + part[3][k];
    metrics[2 * blockIdx.x] = static_cast<float>(tot[0] / tot[1]);
    metrics[2 * blockIdx.x + 1] = with_star ? static_cast<float>(tot[2] / tot[3]) : -1.f;
}

// ---- variant table for stage 1 --------------------------------------------------------------------------------------
// each variant is built twice, for phi = identity and phi = sigmoid: every lane forms the residual of every row, and the kernels
// bound by vector-ALU issue would pay for evaluating both forms and selecting one
#define CR_V(XD, VEC, TS, K, R)                                                                         \
    {XD, VEC, TS, K, R, (TS < 256 ? 256 / TS : 1),                                                      \
     {reinterpret_cast<const void *>(&partial_grads_kernel<XD, VEC, TS, K, R, false>),                  \
      reinterpret_cast<const void *>(&partial_grads_kernel<XD, VEC, TS, K, R, true>)}}
#define CR_VB(XD, VEC, TS, K, R)                                                                        \
    {XD, VEC, TS, K, R, (TS < 256 ? 256 / TS : 1),                                                      \
     {reinterpret_cast<const void *>(&partial_grads_kernel<XD, VEC, TS, K, R, false>),                  \
      reinterpret_cast<const void *>(&partial_grads_kernel<XD, VEC, TS, K, R, true>)},                  \
     {reinterpret_cast<const void *>(&partial_grads_kernel<XD, VEC, TS, K, R, false, true>),            \
      reinterpret_cast<const void *>(&partial_grads_kernel<XD, VEC, TS, K, R, true, true>)}}
// one variant per exact chunk count K = ceil(row chunks / team size); R rows in flight chosen so a thread holds about 16-24 chunks
const Stage1Variant kVariants[] = {
    // fp32, chunks of 4 columns (4 registers per chunk)
    CR_V(0, 4, 64, 1, 8), CR_V(0, 4, 64, 2, 8), CR_V(0, 4, 64, 3, 4), CR_V(0, 4, 64, 4, 4),
    CR_V(0, 4, 256, 2, 8), CR_V(0, 4, 256, 3, 4), CR_V(0, 4, 256, 4, 4), CR_V(0, 4, 256, 5, 4),
    CR_V(0, 4, 256, 6, 3), CR_V(0, 4, 256, 7, 2), CR_V(0, 4, 256, 8, 2), CR_V(0, 4, 256, 9, 2),
    CR_V(0, 4, 256, 10, 2), CR_V(0, 4, 256, 11, 2), CR_V(0, 4, 256, 12, 2),
    CR_V(0, 4, 1024, 4, 2), CR_V(0, 4, 1024, 5, 1), CR_V(0, 4, 1024, 6, 1),
    // bf16, chunks of 8 columns: they widen to eight accumulators each, so a thread can hold half as many
    // (the one-wavefront teams, bound by vector-ALU issue, also come with buffer loads for rows that start on 4-byte boundaries)
    CR_VB(1, 8, 64, 1, 8), CR_VB(1, 8, 64, 2, 4), CR_VB(1, 8, 64, 3, 4), CR_VB(1, 8, 64, 4, 2),
    CR_V(1, 8, 256, 2, 4), CR_V(1, 8, 256, 3, 4), CR_V(1, 8, 256, 4, 2), CR_V(1, 8, 256, 5, 2),
    CR_V(1, 8, 256, 6, 2), CR_V(1, 8, 1024, 2, 2), CR_V(1, 8, 1024, 3, 1),
    // rows shorter than one wide chunk: one column per lane
    CR_V(0, 1, 64, 1, 8), CR_V(1, 1, 64, 1, 8),
};

// every-row-once kernels: threads that share a row, chunks per thread, rows per step, threads per workgroup
#define CR_O(XD, VEC, LPR, K, R, WAVES)                                                                 \
    {XD, VEC, LPR, K, WAVES * R * (64 / LPR), WAVES * 64, 2,                                            \
     {reinterpret_cast<const void *>(&rows_once_kernel<XD, VEC, LPR, K, R, WAVES, false>),              \
      reinterpret_cast<const void *>(&rows_once_kernel<XD, VEC, LPR, K, R, WAVES, true>)}}
#define CR_OT(XD, VEC, TS, K, R, PF)                                                                    \
    {XD, VEC, TS, K, R, TS, XD == 1 && TS == 128 ? 2 : 1,                                               \
     {reinterpret_cast<const void *>(&rows_once_team_kernel<XD, VEC, TS, K, R, PF, false, false>),      \
      reinterpret_cast<const void *>(&rows_once_team_kernel<XD, VEC, TS, K, R, PF, false, true>)}}
#define CR_OW(XD, VEC, K, PF)                                                                           \
    {XD, VEC, 512, K, 1, 512, 1,                                                                        \
     {reinterpret_cast<const void *>(&rows_once_team_kernel<XD, VEC, 512, K, 1, PF, true, false>),      \
      reinterpret_cast<const void *>(&rows_once_team_kernel<XD, VEC, 512, K, 1, PF, true, true>)}}
const OnceVariant kOnceVariants[] = {
    // fp32: up to 256 chunks (1024 columns) a wavefront or a part of one per row ...
    CR_O(0, 4, 2, 1, 4, 4), CR_O(0, 4, 4, 1, 4, 4), CR_O(0, 4, 8, 1, 4, 4), CR_O(0, 4, 16, 1, 4, 4), CR_O(0, 4, 32, 1, 4, 4),
    CR_O(0, 4, 64, 1, 4, 4), CR_O(0, 4, 64, 2, 4, 4), CR_O(0, 4, 64, 3, 2, 4), CR_O(0, 4, 64, 4, 2, 4),
    // ... then two wavefronts up to 512, four up to 1792, eight up to 6144 chunks (more chunks per thread would leave no room for the
    // next step; 60 000 x 1500: 59 us with two wavefronts, 63 with four, a quarter of whose second chunks lie past the row)
    CR_OT(0, 4, 128, 3, 4, true), CR_OT(0, 4, 128, 4, 4, true), CR_OT(0, 4, 256, 3, 4, true), CR_OT(0, 4, 256, 4, 2, true),
    CR_OT(0, 4, 256, 5, 2, true), CR_OT(0, 4, 256, 6, 2, true), CR_OT(0, 4, 256, 7, 2, true),
    CR_OT(0, 4, 512, 4, 2, true), CR_OT(0, 4, 512, 5, 2, true), CR_OT(0, 4, 512, 6, 1, true),
    CR_OT(0, 4, 512, 7, 1, true), CR_OT(0, 4, 512, 8, 1, true), CR_OT(0, 4, 512, 9, 1, true),
    CR_OT(0, 4, 512, 10, 1, false), CR_OT(0, 4, 512, 11, 1, false), CR_OT(0, 4, 512, 12, 1, false),
    // bf16: the same, a chunk widening to eight accumulators
    CR_O(1, 8, 2, 1, 4, 4), CR_O(1, 8, 4, 1, 4, 4), CR_O(1, 8, 8, 1, 4, 4), CR_O(1, 8, 16, 1, 4, 4), CR_O(1, 8, 32, 1, 4, 4),
    CR_O(1, 8, 64, 1, 4, 4), CR_O(1, 8, 64, 2, 2, 4), CR_O(1, 8, 64, 3, 2, 4), CR_O(1, 8, 64, 4, 2, 4),
    // (rows of an odd number of columns start on any 2-byte boundary, where 16-byte loads take two trips: two smaller workgroups per
    // unit hide that better, 3 GB of 3001 columns 509 against 785 us, of 6001 columns 517 against 662)
    CR_OT(1, 8, 128, 3, 4, true), CR_OT(1, 8, 128, 4, 2, true), CR_OT(1, 8, 128, 5, 2, true),
    CR_OT(1, 8, 128, 6, 2, true),
    CR_OT(1, 8, 256, 2, 4, true), CR_OT(1, 8, 256, 3, 2, true), CR_OT(1, 8, 256, 4, 2, true),
    CR_OT(1, 8, 512, 3, 1, true), CR_OT(1, 8, 512, 4, 1, true), CR_OT(1, 8, 512, 5, 1, true),
    CR_OT(1, 8, 512, 6, 1, true),
    // rows shorter than one wide chunk: one column per lane
    CR_O(0, 1, 4, 1, 4, 4), CR_O(1, 1, 8, 1, 4, 4),
};
// wide rows whose weights fit LDS
const OnceVariant kOnceVariantsWide[] = {
    CR_OW(0, 4, 13, false), CR_OW(0, 4, 14, false), CR_OW(0, 4, 15, false), CR_OW(0, 4, 16, false), CR_OW(0, 4, 17, false),
    CR_OW(1, 8, 7, true), CR_OW(1, 8, 8, false), CR_OW(1, 8, 9, false),
};
// several workgroups per row
#define CR_OC(XD, VEC, K, R)                                                                            \
    {XD, VEC, K, R, 0, 0,                                                                               \
     {reinterpret_cast<const void *>(&rows_once_crew_kernel<XD, VEC, K, R, false>),                     \
      reinterpret_cast<const void *>(&rows_once_crew_kernel<XD, VEC, K, R, true>)}}
const CrewVariant kCrewVariants[] = {
    CR_OC(0, 4, 2, 4), CR_OC(0, 4, 3, 2), CR_OC(0, 4, 4, 2), CR_OC(1, 8, 2, 4), CR_OC(1, 8, 3, 2),
};
// one row per wavefront or less, sixteen wavefronts: for launches of a few workgroups that each have a whole slab range to do
const OnceVariant kOnceVariants16[] = {
    CR_O(0, 4, 2, 1, 4, 16), CR_O(0, 4, 4, 1, 4, 16), CR_O(0, 4, 8, 1, 4, 16), CR_O(0, 4, 16, 1, 4, 16), CR_O(0, 4, 32, 1, 4, 16),
    CR_O(0, 4, 64, 1, 4, 16), CR_O(1, 8, 2, 1, 4, 16), CR_O(1, 8, 4, 1, 4, 16), CR_O(1, 8, 8, 1, 4, 16), CR_O(1, 8, 16, 1, 4, 16),
    CR_O(1, 8, 32, 1, 4, 16), CR_O(1, 8, 64, 1, 4, 16), CR_O(0, 1, 4, 1, 4, 16), CR_O(1, 1, 8, 1, 4, 16),
};

// columns per chunk: the 16-byte width unless the row is shorter than that
int stage1_chunk_width(int x_dtype, int64_t d)
{
    const int wide = (x_dtype == 1) ? 8 : 4;
    return d >= wide ? wide : 1;
}

}  // namespace

const Stage1Variant *select_stage1(int x_dtype, int64_t d)
{
    const int vec = stage1_chunk_width(x_dtype, d);
    const int64_t nq = (d + vec - 1) / vec;
    // smallest team that covers the row with an available chunk count; the kernel needs K = ceil(nq / team size) exactly
    for (int ts : {64, 256, 1024}) {
        const int64_t k = (nq + ts - 1) / ts;
        for (const Stage1Variant &v : kVariants)
            if (v.xd == x_dtype && v.vec == vec && v.team_size == ts && v.k == k) return &v;
    }
    return nullptr;
}

namespace {
const OnceVariant *find_once(const OnceVariant *begin, const OnceVariant *end, int x_dtype, int64_t d)
{
    const int vec = stage1_chunk_width(x_dtype, d);
    const int64_t nq = (d + vec - 1) / vec;
    for (const OnceVariant *v = begin; v != end; ++v) {
        if (v->xd != x_dtype || v->vec != vec || (x_dtype == 1 && v->threads_per_row == 128 && d % 2 == 0)) continue;
        // listed from narrow to wide: the first that covers the row.  K is exact, so that only a thread's last chunk can lie past it
        if (v->threads_per_row <= 64 ? nq <= static_cast<int64_t>(v->threads_per_row) * v->k
                                     : v->k == (nq + v->threads_per_row - 1) / v->threads_per_row) return v;
    }
    return nullptr;
}
}  // namespace

const OnceVariant *select_once(int x_dtype, int64_t d) { return find_once(std::begin(kOnceVariants), std::end(kOnceVariants), x_dtype, d); }
const OnceVariant *select_once_wide(int x_dtype, int64_t d) { return find_once(std::begin(kOnceVariantsWide), std::end(kOnceVariantsWide), x_dtype, d); }
const OnceVariant *select_once_whole(int x_dtype, int64_t d)
{
    const OnceVariant *v = find_once(std::begin(kOnceVariants16), std::end(kOnceVariants16), x_dtype, d);
    return v ? v : select_once(x_dtype, d);
}

// Of the numbers of workgroups that can share the row: full dies count most, then slices that fill their threads' chunks, then few rows
// per step against them.  400 MB, us with sums, by workgroups (share of the chunks in use), two passes: bf16 37 000 columns K = 2 x 6
// (0.86) 79.0, K = 3 x 4 (0.86) 84.6, 131; 50 008 K = 2 x 8 (0.87) 79.0, x 7 (1.00) 80.8, K = 3 x 5 (0.93) 87.3, 131; 80 001 K = 3 x 8 (0.93)
// 95.0, K = 2 x 12 (0.93) 108, 144; 100 000 K = 2 x 16 (0.87) 84.6, x 14 (1.00) 86.0, 134; fp32 40 001 K = 3 x 8 (0.93) 75.8, K = 2 x 12 (0.93)
// 77.9, K = 4 x 6 (0.93) 80.3, 128; 60 000 K = 4 x 10 (0.84) 85.2, x 9 (0.93) 89.9, K = 3 x 16 (0.70) 91.8, 125.
bool select_crew(int x_dtype, int64_t d, int units, CrewVariant *v)
{
    const int vec = stage1_chunk_width(x_dtype, d), on_die = units / 8 > 0 ? units / 8 : 1;
    const int64_t nq = (d + vec - 1) / vec;
    double best = 0.0;
    for (int members = 2; members <= kCrewMembers && members <= on_die; ++members) {
        const int64_t per = (nq + members - 1) / members;
        for (const CrewVariant &c : kCrewVariants) {
            if (c.xd != x_dtype || c.vec != vec || c.k != (per + kCrewThreads - 1) / kCrewThreads) continue;
            const double used = static_cast<double>(on_die / members * members) / on_die;
            const double score = used * used * static_cast<double>(per) / (c.k * kCrewThreads) * (x_dtype == 1 && c.k > 2 ? 0.85 : 1.0);
            if (score <= best) continue;
            best = score;
            *v = c;
            v->members = members;
        }
    }
    return best > 0.0;
}

// Steps whose slots are kept: all of a part's, so that a member that starts late finds every answer (4 000 rows: 32 steps, 512 KB of slots), or
// the last 1 024 (some 2 ms of work).
int crew_ring_steps(const CrewVariant &v, int64_t longest_part)
{
    int steps = 16;
    while (steps < 1024 && static_cast<int64_t>(steps) * v.rows_per_step < longest_part) steps *= 2;
    return steps;
}
int64_t crew_exchange_words(const CrewVariant &v) { return static_cast<int64_t>(v.ring_steps) * v.members * v.rows_per_step; }

hipError_t launch_rows_once_crew(const CrewVariant &v, const void *X, const float *y, const float *w, const DevRun *parts, int num_parts,
                                 const DevRun *runs, const int32_t *dst, float *rows, int64_t d, int logistic, bool stream_past_caches,
                                 uint64_t *slots, uint32_t *state, int patience, hipStream_t stream)
{
    int di = static_cast<int>(d), nq = static_cast<int>((d + v.vec - 1) / v.vec), members = v.members, ring_steps = v.ring_steps;
    void *args[] = {&X, &y, &w, &parts, &runs, &dst, &rows, &di, &nq, &logistic, &num_parts, &members, &slots, &ring_steps, &state, &patience};
    return hipLaunchKernel(v.fn[stream_past_caches ? 1 : 0], dim3((num_parts + 7) / 8 * 8 * members), dim3(kCrewThreads + 64), args, 0, stream);
}

hipError_t launch_rows_once(const OnceVariant &v, const void *X, const float *y, const float *w, const DevRun *parts, int num_parts,
                            const DevRun *runs, const int32_t *dst, float *rows, int64_t d, int logistic, bool stream_past_caches,
                            hipStream_t stream)
{
    int di = static_cast<int>(d);
    int nq = static_cast<int>((d + v.vec - 1) / v.vec);
    void *args[] = {&X, &y, &w, &parts, &runs, &dst, &rows, &di, &nq, &logistic};
    return hipLaunchKernel(v.fn[stream_past_caches ? 1 : 0], dim3(num_parts), dim3(v.block), args, 0, stream);
}

hipError_t launch_partial_grads(const Stage1Variant &v, const void *X, const float *y, const float *w, const DevPiece *pieces,
                                const int32_t *team_piece_begin, int num_teams, float *rows, int64_t d, int logistic,
                                bool rows_as_buffers, hipStream_t stream)
{
    int di = static_cast<int>(d);
    int nq = static_cast<int>((d + v.vec - 1) / v.vec);
    void *args[] = {&X, &y, &w, &pieces, &team_piece_begin, &num_teams, &rows, &di, &nq};
    const int tpb = v.teams_per_block();
    dim3 grid((num_teams + tpb - 1) / tpb), block(v.block());
    const void *fn = rows_as_buffers && v.fn_buffers[0] ? v.fn_buffers[logistic ? 1 : 0] : v.fn[logistic ? 1 : 0];
    return hipLaunchKernel(fn, grid, block, args, 0, stream);
}

namespace {
template <int XD, int VEC>
hipError_t launch_wide(const void *X, const float *y, const float *w, const DevPiece *pieces, int num_pieces, float *residuals,
                       float *rows, int64_t d, int logistic, hipStream_t stream)
{
    const int nq = static_cast<int>((d + VEC - 1) / VEC);
    const int di = static_cast<int>(d);
    if (rows == nullptr)
        residuals_kernel<XD, VEC><<<num_pieces, 256, 0, stream>>>(X, y, w, pieces, residuals, di, nq, logistic);
    else
        xt_residuals_kernel<XD, VEC><<<dim3((nq + 256 * kWideChunks - 1) / (256 * kWideChunks), num_pieces), 256, 0, stream>>>(
            X, pieces, residuals, rows, di, nq);
    return hipGetLastError();
}

hipError_t dispatch_wide(int x_dtype, const void *X, const float *y, const float *w, const DevPiece *pieces, int num_pieces,
                         float *residuals, float *rows, int64_t d, int logistic, hipStream_t stream)
{
    if (x_dtype == 0) return launch_wide<0, 4>(X, y, w, pieces, num_pieces, residuals, rows, d, logistic, stream);
    return launch_wide<1, 8>(X, y, w, pieces, num_pieces, residuals, rows, d, logistic, stream);
}
}  // namespace

hipError_t launch_residuals(int x_dtype, const void *X, const float *y, const float *w, const DevPiece *pieces, int num_pieces,
                            float *residuals, int64_t d, int logistic, hipStream_t stream)
{
    return dispatch_wide(x_dtype, X, y, w, pieces, num_pieces, residuals, nullptr, d, logistic, stream);
}

hipError_t launch_xt_residuals(int x_dtype, const void *X, const DevPiece *pieces, int num_pieces, const float *residuals, float *rows,
                               int64_t d, hipStream_t stream)
{
    return dispatch_wide(x_dtype, X, nullptr, nullptr, pieces, num_pieces, const_cast<float *>(residuals), rows, d, 0, stream);
}

namespace {
template <int XD, int VEC>
hipError_t wide_once(const void *X, const float *y, const float *w, float *residuals, int64_t m, const DevRun *parts, int num_parts, const DevRun *runs,
                     const int32_t *dst, float *rows, int64_t d, int logistic, int64_t cached_from, int units, hipStream_t stream)
{
    const int nq = static_cast<int>((d + VEC - 1) / VEC), di = static_cast<int>(d);
    auto residuals_of = [&](auto r) {
        constexpr int R = decltype(r)::value;
        wide_residuals_kernel<XD, VEC, R><<<static_cast<unsigned>((m + R - 1) / R), 512, 0, stream>>>(X, y, w, residuals, m, di, nq, logistic, cached_from);
    };
    // the most rows per workgroup that still leave the chip nearly two workgroups per compute unit
    const int64_t enough = 2 * static_cast<int64_t>(units) * 7 / 8;
    if (m >= 8 * enough) residuals_of(std::integral_constant<int, 8>{});
    else if (m >= 4 * enough) residuals_of(std::integral_constant<int, 4>{});
    else if (m >= 2 * enough) residuals_of(std::integral_constant<int, 2>{});
    else residuals_of(std::integral_constant<int, 1>{});
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    wide_xt_kernel<XD, VEC><<<dim3((nq + 255) / 256, num_parts), 256, 0, stream>>>(X, residuals, parts, runs, dst, rows, di, nq, cached_from);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_wide_once(int x_dtype, const void *X, const float *y, const float *w, float *residuals, int64_t m, const DevRun *parts, int num_parts,
                            const DevRun *runs, const int32_t *dst, float *rows, int64_t d, int logistic, int64_t cached_from, int units,
                            hipStream_t stream)
{
    if (x_dtype == 0) return wide_once<0, 4>(X, y, w, residuals, m, parts, num_parts, runs, dst, rows, d, logistic, cached_from, units, stream);
    return wide_once<1, 8>(X, y, w, residuals, m, parts, num_parts, runs, dst, rows, d, logistic, cached_from, units, stream);
}

hipError_t launch_sum_rows(float *rows, const DevSum *sums, int num_sums, int64_t summed, const int32_t *dst, int64_t d, hipStream_t stream)
{
    constexpr int kMaxGridY = 65535;
    const int nq = static_cast<int>(d >= 4 ? (d + 3) / 4 : d);
    // A wavefront for all rows of a sum where there are wavefronts enough to make up for the longer chain: 48 times the rows of a sum.  us, a
    // workgroup / a wavefront, by wavefronts per row of a sum: (2,12), s = 1, 5 001 columns (390) 9.9 / 7.8, 50 008 bf16 33.6 / 17.4; (3,6), s = 2,
    // 20 001 31.7 / 21.3; (2,4) 50 008 bf16 (700) 11.2 / 8.0; (3,4) 20 001 (190) 15.0 / 12.4, 6 500 (62) 8.4 / 8.3, 5 001 (48) 7.9 / 8.2; (2,4) 20 001
    // (34) 10.6 / 12.0, 5 001 (9) 7.0 / 10.0; (3,6) 1 024 (17) 7.5 / 10.3; (1,10), s = 4, 20 001 (6) 9.5 / 9.9
    const int64_t wavefronts = static_cast<int64_t>((nq + 63) / 64) * num_sums;
    const bool few = d >= 4 && num_sums > 0 && wavefronts >= 256 && wavefronts * num_sums > 48 * summed;
    for (int lo = 0; lo < num_sums; lo += kMaxGridY) {
        const dim3 grid((nq + 63) / 64, num_sums - lo < kMaxGridY ? num_sums - lo : kMaxGridY);
        if (few) {
            sum_few_rows_kernel<<<dim3((nq + 255) / 256, grid.y), 256, 0, stream>>>(rows, sums + lo, dst, d, nq);
            continue;
        }
        if (d >= 4) sum_rows_kernel<4><<<grid, 512, 0, stream>>>(rows, sums + lo, dst, d, nq);
        else sum_rows_kernel<1><<<grid, 512, 0, stream>>>(rows, sums + lo, dst, d, nq);
    }
    return hipGetLastError();
}

template <int VEC, int C, int BS, int U, bool NTS, typename acc_t>
static hipError_t launch_encode_shape(const float *G, float *M, const EncProgram &prog, int num_sub, int L, int64_t d, hipStream_t stream)
{
    const int nq = static_cast<int>((d + VEC - 1) / VEC);
    const dim3 grid((nq + BS * C - 1) / (BS * C), num_sub), block(BS);
    if (L <= 1) encode_kernel<VEC, 1, C, BS, U, NTS, acc_t><<<grid, block, 0, stream>>>(G, M, prog, d, nq);
    else if (L == 2) encode_kernel<VEC, 2, C, BS, U, NTS, acc_t><<<grid, block, 0, stream>>>(G, M, prog, d, nq);
    else if (L == 3) encode_kernel<VEC, 3, C, BS, U, NTS, acc_t><<<grid, block, 0, stream>>>(G, M, prog, d, nq);
    else if constexpr (C == 1) {                         // deeper trees only in the narrow shape (the wide one would spill)
        if (L == 4) encode_kernel<VEC, 4, C, BS, U, NTS, acc_t><<<grid, block, 0, stream>>>(G, M, prog, d, nq);
        else encode_kernel<VEC, kMaxLevels, C, BS, U, NTS, acc_t><<<grid, block, 0, stream>>>(G, M, prog, d, nq);
    } else return hipErrorInvalidValue;
    return hipGetLastError();
}

// wide shape once its 8192-chunk workgroups are enough to fill the chip, and only up to 3 levels (registers)
static bool encode_is_wide(int n, int L, int64_t d) { return d >= 4 && ((d + 3) / 4 + 8191) / 8192 * n >= 256 && L <= 3; }

// The rule for one launch of all masks.  A workgroup keeps its 64 chunks of columns for all of them, so that a round of a workgroup per
// compute unit that is less than half full costs as much as a full one, and every next one the more the more slabs there are.  What the
// launch saves is the launches and ramps of each mask.  us a mask, eight masks with gradients of their own, a launch of each kind per mask / one
// launch:
//   one round    (2,12), s = 2, 65 536 columns 25.9 / 17.7; (3,6), s = 2, 32.0 / 26.0; (2,24), s = 1, 61.7 / 53.5
//   two          73 728 columns: (2,8), s = 2 (248 slabs) 17.9 / 13.4; (3,5) (345) 23.8 / 20.9; (2,12), s = 2 (444) 28.4 / 24.5, 77 000 27.5 / 27.8;
//                (2,14), s = 1 (406) 29.7 / 30.8, 67 000 27.8 / 32.0; (2,12), s = 5 (888) 36.0 / 37.1; (2,17) (629) 40.1 / 44.5; 95 000: (2,12), s = 5
//                43.7 / 42.4, (3,6), s = 2 (756) 46.8 / 41.8; 117 706: (2,12), s = 5 51.9 / 49.4, (2,17) 61.1 / 56.0, (3,8), s = 2 (2104) 145 / 149
//   three, four  160 001: (2,8) 29.2 / 26.6; (3,5) 44.2 / 38.9; (2,12), s = 5 69.5 / 70.4; 200 003: s = 2 63.5 / 65.9, s = 5 86.8 / 93.3
//   more         300 001: (3,6), s = 2 130 / 146; 400 001: (2,12), s = 2 122 / 126, s = 5 165 / 177, (2,8) 66.5 / 66.1, (3,4) (148) 44.3 / 42.8;
//                800 001: (3,4) 80.4 / 84.7
//   messages of 256 MB and more   (2,12), s = 1, 600 001 159 / 162; (3,6) 400 001 180 / 196; (2,24) (1176) 160 001 153 / 151.  That line is from when
//                every mask wrote all its messages, 224 / 183, 258 / 229 and 249 / 206: one launch is no longer ahead there, and behind on three levels.
// Up to 32 768 columns a launch per mask needs no copy of programs: (2,24), s = 1, 1 000 columns 16.9 / 29.8.  (Towards 32 768 one launch takes
// the device less, (2,12), s = 2, 16.5 / 12.0, but the host builds its programs.)  A single mask has less to save (and the nodes side by side where
// tree_side_by_side says so): (2,12), s = 2, 117 706 65.6 / 64.9, 200 003 94.3 / 99.7; s = 5, 81 920 58.9 / 64.0; (2,32), s = 1, 40 001 110 / 120.
bool encode_in_steps(const TreeShape &tree, int64_t d, int steps)
{
    if (tree.n > 32 || tree.L > 3 || d <= kTogetherColumns || encode_is_wide(tree.n, tree.L, d)) return false;
    if (tree.n <= 4 || (tree.L == 1 && tree.n * d <= int64_t(1) << 22)) return true;
    constexpr int64_t kUnits = 256;
    const int64_t groups = (d + 255) / 256, messages = static_cast<int64_t>(tree.nodes) * d * 4 / tree.n * (tree.n - tree.s);
    const bool half_empty = groups > kUnits && 2 * groups < 3 * kUnits;
    const int64_t load = tree.slabs * groups;
    if (steps == 1) return groups <= 2 * kUnits && load <= (half_empty ? 160000 : 300000);
    if (groups <= 2 * kUnits && !half_empty) return true;
    return messages >= int64_t(256) << 20 || load <= (4 * groups < 5 * kUnits ? 100000 : 300000);
}

hipError_t launch_encode_steps(const float *G, int64_t G_stride, float *M, const EncProgram &prog, int64_t prog_stride, int steps, int n, int L,
                               float *g, int64_t g_stride, int64_t d, hipStream_t stream)
{
    const int nq = static_cast<int>((d + 3) / 4);
    const unsigned groups = ((nq + 63) / 64 + 7) / 8 * 8, block = 64 * (n < 16 ? n : 16);
    const size_t lds = static_cast<size_t>(2) * n * 4 * 64 * sizeof(float);
    if (L <= 1) encode_steps_kernel<1><<<groups, block, lds, stream>>>(G, G_stride, M, prog, prog_stride, steps, n, g, g_stride, d, nq);
    else if (L == 2) encode_steps_kernel<2><<<groups, block, lds, stream>>>(G, G_stride, M, prog, prog_stride, steps, n, g, g_stride, d, nq);
    else if (L == 3) encode_steps_kernel<3><<<groups, block, lds, stream>>>(G, G_stride, M, prog, prog_stride, steps, n, g, g_stride, d, nq);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_encode(const float *G, float *M, const EncProgram &prog, int num_sub, int L, int64_t d, hipStream_t stream)
{
    if (d >= 4) {
        if (encode_is_wide(num_sub, L, d)) return launch_encode_shape<4, 32, 256, 1, true, float>(G, M, prog, num_sub, L, d, stream);
        return launch_encode_shape<4, 1, 256, 8, false, double>(G, M, prog, num_sub, L, d, stream);
    }
    return launch_encode_shape<1, 1, 256, 8, false, double>(G, M, prog, num_sub, L, d, stream);
}

namespace {
constexpr size_t kTreeLdsBytes = size_t(60) << 10;          // 64 KB with ArgumentTables' copy
static_assert(sizeof(ArgumentTables) <= 3776 && sizeof(DeviceTables) <= 3776 && sizeof(TreeLevels) + sizeof(GradientStep) + sizeof(NodeBits) + 64 <= 320, "4 KB of kernel arguments");

// the nodes of one level-1 sub-tree, or of all of them
TreeLevels tree_levels(int n, int L, bool whole)
{
    TreeLevels t = {};
    t.n = n;
    t.L = L;
    int offset = 0, width = 1, count[kMaxLevels];
    for (int l = 1; l <= L; ++l) {
        t.width[l - 1] = width;
        t.shift[l - 1] = offset;
        count[l - 1] = whole ? width * n : width;
        width *= n;
        offset += width;                                 // a level has n times as many nodes as one sub-tree has of it
    }
    for (int l = L; l >= 1; --l) {
        t.first[l - 1] = t.total;
        t.shift[l - 1] -= t.total;
        t.total += count[l - 1];
    }
    t.leaves = count[L - 1];
    return t;
}

template <int VEC, int B> bool tree_fits(const TreeLevels &tree) { return TreeLds<VEC, B>::bytes(tree.total, tree.leaves) <= kTreeLdsBytes; }

// Threads of a workgroup that has `nodes` nodes and B lanes for each: the more nodes have a team of their own the fewer fetches follow
// one another, as long as the workgroups that LDS leaves room for are on the chip at once (us of the kernel, 256 threads / more): (3,6), s = 2,
// 1 024 columns 8.2 / 6.5 (704), 40 000, three workgroups per unit for their LDS, 28.0 / 24.6 (384); (3,4) 50 008, five, 10.6 / 12.3 (512);
// encode and decode together, (2,12), s = 2, 512 / 1 024: 12 288 columns 12.0 / 10.0, 24 576, two per unit, 14.1 / 16.8.
// Fewer threads where there are fewer nodes: (1,64) 16 384 columns 10.8 (256) / 7.5 (64).
template <int B> int tree_threads(int nodes, int groups, size_t lds)
{
    constexpr int kUnits = 256, kWavefronts = B == 64 ? 20 : 16;      // of a compute unit, by their registers
    const int resident = std::max(1, std::min((groups + kUnits - 1) / kUnits, static_cast<int>((size_t(160) << 10) / lds)));
    const int teams = std::min(1024, std::max(256, kWavefronts / resident * 64)) / B, rounds = (nodes + teams - 1) / teams;
    return ((nodes + rounds - 1) / rounds * B + 63) / 64 * 64;         // no more than it takes for as few rounds
}

template <int VEC, int B, typename TABLES>
hipError_t launch_tree_shape(const float *G, float *M, const TABLES &tables, const NodeBits &stored, TreeLevels tree, int64_t d, hipStream_t stream)
{
    const int nq = static_cast<int>((d + VEC - 1) / VEC), groups = (nq + B - 1) / B;
    const size_t lds = TABLES::kLdsBytes + TreeLds<VEC, B>::bytes(tree.total, tree.leaves);
    tree.threads = tree_threads<B>(tree.total, groups * tree.n, lds);
    tree_kernel<VEC, B><<<dim3(groups, tree.n), tree.threads, lds, stream>>>(G, M, tables, stored, tree, d, nq);
    return hipGetLastError();
}

template <typename TABLES>
hipError_t launch_tree(const float *G, float *M, const TABLES &tables, const NodeBits &stored, int n, int L, int64_t d, hipStream_t stream)
{
    const TreeLevels tree = tree_levels(n, L, false);
    if (d < 4) return launch_tree_shape<1, 16>(G, M, tables, stored, tree, d, stream);
    // 64 chunks: the team is a wavefront, whose tables and base addresses are scalars, and pieces of a slab are four times as long.  Short
    // vectors only where every node then has a wavefront (us, 16 chunks / 64: (4,2), 15 nodes, 300 columns 6.9 / 5.2, 16 384 7.2 / 5.7; (2,12), 13,
    // 2 048 5.5 / 5.0, 12 288 9.8 / 8.4; (3,5), s = 1, 31 nodes, 1 024 6.3 / 7.0, 4 096 7.1 / 7.1, 12 288 9.9 / 8.1; (3,4), 21, 16 384 7.6 / 6.3;
    // (2,17) 6 500 14.5 / 8.7; (1,64) 8 192 5.7 / 3.5, 32 768 14.5 / 6.9)
    if ((tree.total <= 16 || d > 3072) && tree_fits<4, 64>(tree)) return launch_tree_shape<4, 64>(G, M, tables, stored, tree, d, stream);
    return launch_tree_shape<4, 16>(G, M, tables, stored, tree, d, stream);
}

template <int VEC, int B, typename TABLES>
hipError_t launch_tree_decode_shape(const float *G, float *M, const TABLES &tables, const NodeBits &stored, TreeLevels tree, float *g,
                                    const GradientStep &step, int64_t d, hipStream_t stream)
{
    const int nq = static_cast<int>((d + VEC - 1) / VEC), groups = (nq + B - 1) / B;
    const size_t lds = TABLES::kLdsBytes + TreeLds<VEC, B>::bytes(tree.total, tree.leaves);
    tree.threads = tree_threads<B>(tree.total, groups, lds);
    tree_decode_kernel<VEC, B><<<groups, tree.threads, lds, stream>>>(G, M, tables, stored, tree, g, step, d, nq);
    return hipGetLastError();
}

// Chunks of columns per workgroup that has the whole tree.  Four where the nodes are more than teams of eight lanes and the vector is short
// (us, eight / four: (2,12), s = 2, 10 columns 6.3 / 5.5, 1 024 7.2 / 6.6, 2 048 7.2 / 6.8, 4 096 7.4 / 7.7; (3,5) 1 024 8.2 / 7.5, 4 096 8.5 / 7.9,
// 6 000 9.0 / 10.0).
int tree_decode_chunks(const TreeLevels &tree, int64_t d)
{
    if (d > kTogetherNarrowColumns && tree_fits<4, 16>(tree)) return 16;
    return d >= 4 && d <= 2048 && tree.total * 8 > 1024 ? 4 : 8;
}

template <typename TABLES>
hipError_t launch_tree_decode(const float *G, float *M, const TABLES &tables, const NodeBits &stored, int n, int L, float *g,
                              const GradientStep &step, int64_t d, hipStream_t stream)
{
    const TreeLevels tree = tree_levels(n, L, true);
    if (d < 4) return launch_tree_decode_shape<1, 8>(G, M, tables, stored, tree, g, step, d, stream);
    const int chunks = tree_decode_chunks(tree, d);
    if (chunks == 16) return launch_tree_decode_shape<4, 16>(G, M, tables, stored, tree, g, step, d, stream);
    if (chunks == 4) return launch_tree_decode_shape<4, 4>(G, M, tables, stored, tree, g, step, d, stream);
    return launch_tree_decode_shape<4, 8>(G, M, tables, stored, tree, g, step, d, stream);
}
}  // namespace

// Up to 32 768 columns the nodes side by side are ahead of a walk on every tree.  Beyond, it depends on what the walk's program costs, on
// the wavefronts that the LDS of 64 chunks leaves in flight (32 KB: five workgroups per compute unit), and on whether slabs and
// messages in use leave room in the last-level cache, past which the walk reads.  us of a whole iteration on few rows, walk / side by side:
//   a copy each      32 KB        (2,12), s = 2, 40 001 columns 75.1 / 53.7, 98 304 (188 MB in use) 136 / 129, 117 706 (225 MB) 172 / 173; s = 5,
//                                 81 920 (190 MB) 139 / 129; (3,4) 65 536 53.4 / 49.4, 160 001 (106 MB) 101 / 95; (2,8) 117 706 (108 MB)
//                                 113 / 105, 160 001 (146 MB) 149 / 155; (1,64) 98 304 75.3 / 47.4
//                    60 KB        (3,6), s = 2, 49 152 (127 MB) 118 / 102, 65 536 (169 MB) 147 / 150; (3,5), s = 1, 73 728 (112 MB) 108 / 106, 98 304
//                                 (150 MB) 137 / 142; s = 4, 65 536 92.1 / 79.1
//                    more         (5,2) 49 152 44.2 / 39.0, 57 344 46.8 / 46.6; (4,3) 40 001 65.1 / 61.9, 57 344 72.5 / 72.6
//   16 in a copy     21 KB        (2,12), s = 2, 73 728 (141 MB) 86.3 / 85.5, 98 304 (188 MB) 111 / 119; s = 5, 57 344 (133 MB) 84.4 / 83.5, 65 536 (152 MB)
//                                 95.9 / 103; (2,4) 49 152 26.0 / 23.4, 160 001 47.8 / 46.9; (1,10) 65 536 28.4 / 25.1; (2,17) 40 001 (134 MB) 123 / 121
//                    32 KB        (3,4) 40 001 42.1 / 38.6, 81 920 57.3 / 57.3, 98 304 63.5 / 66.5; (4,2) 73 728 31.3 / 30.6
//                    more         (3,6) 40 001 85.2 / 83.1, 57 344 107 / 119; (3,5), s = 4, 40 001 55.7 / 55.7, 65 536 74.6 / 79.1; (5,2) 40 001 41.9 / 37.6;
//                                 (4,3) 59.9 / 60.4; (6,2) 54.8 / 55.6
//   launches         10 KB        (2,4) 40 001 20.6 / 16.0, 160 001 18.9 / 15.5; (1,64) 160 001 48.4 / 40.6
//                    32 KB        (2,8) 65 536 21.1 / 17.0, 81 920 19.4 / 20.2; (2,12), s = 5, 40 001 26.2 / 23.3, 81 920 39.0 / 38.4; beside the
//                                 arguments' copy (3,4), 31 KB, 65 536 20.0 / 16.7, 73 728 19.4 / 19.9
//                    60 KB        (3,5), s = 4, 40 001 19.6 / 17.3, 65 536 19.2 / 20.0; s = 1, 40 001 25.1 / 23.5, 57 344 24.1 / 27.2
//                    more         (4,3) 33 001 21.7 / 24.2
bool tree_side_by_side(const TreeShape &tree, int64_t d, Otherwise otherwise)
{
    const TreeLevels sub = tree.nodes <= NodeCoefs::kNodes ? tree_levels(tree.n, tree.L, false) : TreeLevels();
    if (tree.nodes > NodeCoefs::kNodes || d > kTreeColumns || !tree_fits<4, 16>(sub)) return false;
    if (d <= kTreeNarrowColumns) return true;
    const size_t lds = TreeLds<4, 64>::bytes(sub.total, sub.leaves), kb = size_t(1) << 10;
    const int64_t in_use = (tree.slabs + tree.nodes) * d * 4 / tree.n * (tree.n - tree.s), mb = int64_t(1) << 20;
    switch (otherwise) {
    case Otherwise::kBatch:
        return lds <= 32 * kb ? in_use <= 141 * mb && (lds <= 21 * kb || d <= 81920) : d <= 40960;
    case Otherwise::kLaunches:
        return lds <= 10 * kb || (lds <= 30 * kb && d <= 81920) || (lds <= 32 * kb && d <= 65536) || (tree_fits<4, 64>(sub) && d <= 40960);
    case Otherwise::kCopy:
        if (lds <= 32 * kb) return in_use <= 190 * mb && (d <= 131072 || in_use <= 120 * mb);
        return tree_fits<4, 64>(sub) ? in_use <= 130 * mb : d <= 49152;
    }
    return false;
}

// From 8 192 columns on, where the whole tree's messages do not fit LDS for 16 chunks, the launch has twice the workgroups, of eight chunks,
// each with the whole chain of a deep tree; on two levels that still pays, or costs little.  us of encode and decode apart / together: (3,6), s = 2,
// 4 096 columns 10.0 / 9.8, 8 195 11.4 / 14.3, 16 384 15.0 / 16.4, 32 768 23.3 / 35.9; (2,17), s = 1, 8 192 13.3 / 11.6, 16 384 17.1 / 16.8, 24 576
// 20.9 / 22.5; (2,19) 8 192 15.0 / 12.6, 16 384 18.8 / 19.0, 32 768 29.9 / 36.3.  Where they fit: (6,2) 32 768 18.6 / 17.1; (2,8), s = 2, 32 768
// 11.6 / 11.2; (1,64) 32 768 19.3 / 11.8; (2,12), s = 2, 12 288 10.7 / 10.3, 20 480 12.8 / 15.3, 32 768 16.1 / 16.6.  (An encode alone has become
// faster than when the line at 32 768 columns was drawn: trees of 150 nodes and more on two levels are up to 20 % behind from 20 000 columns on.)
bool tree_and_decode_together(const TreeShape &tree, int64_t d)
{
    const TreeLevels whole = tree.nodes <= NodeCoefs::kNodes ? tree_levels(tree.n, tree.L, true) : TreeLevels();
    if (d > kTogetherColumns || !tree_side_by_side(tree, d, Otherwise::kCopy) || !tree_fits<4, 8>(whole)) return false;
    return d <= kTogetherNarrowColumns || tree.L <= 2 || tree_fits<4, 16>(whole);
}

int tree_decode_groups(int n, int L, int64_t d)
{
    const int64_t chunks = d < 4 ? d : (d + 3) / 4;
    const int per = tree_decode_chunks(tree_levels(n, L, true), d);
    return static_cast<int>((chunks + per - 1) / per);
}

namespace {
// f(tables), with as short an argument as they fit
template <typename F> hipError_t with_short(const DeviceTables &tables, int nodes, F f)
{
    if (nodes > SmallDeviceTables::kNodes) return f(tables);
    SmallDeviceTables small = {tables.node_begin, tables.slab_coef, {}};
    std::copy(tables.coefs.a, tables.coefs.a + nodes, small.coefs.a);
    return f(small);
}
template <typename F> hipError_t with_short(const ArgumentTables &tables, int, F f)
{
    if (tables.used > SmallArgumentTables::kWords) return f(tables);
    SmallArgumentTables small = {tables.at_begin, tables.at_coef, tables.at_slab, tables.used, {}};
    std::copy(tables.word, tables.word + tables.used, small.word);
    return f(small);
}
int nodes_of(int n, int L)
{
    int nodes = 0;
    for (int l = 0; l < L; ++l) nodes = (nodes + 1) * n;
    return nodes;
}
}  // namespace

hipError_t launch_tree_encode(const float *G, float *M, const DeviceTables &tables, const NodeBits &stored, int n, int L, int64_t d, hipStream_t stream)
{
    return with_short(tables, nodes_of(n, L), [&](const auto &t) { return launch_tree(G, M, t, stored, n, L, d, stream); });
}

hipError_t launch_tree_encode(const float *G, float *M, const ArgumentTables &tables, const NodeBits &stored, int n, int L, int64_t d, hipStream_t stream)
{
    return with_short(tables, nodes_of(n, L), [&](const auto &t) { return launch_tree(G, M, t, stored, n, L, d, stream); });
}

hipError_t launch_tree_encode_decode(const float *G, float *M, const DeviceTables &tables, const NodeBits &stored, int n, int L, float *g,
                                     const GradientStep &step, int64_t d, hipStream_t stream)
{
    return with_short(tables, nodes_of(n, L), [&](const auto &t) { return launch_tree_decode(G, M, t, stored, n, L, g, step, d, stream); });
}

hipError_t launch_tree_encode_decode(const float *G, float *M, const ArgumentTables &tables, const NodeBits &stored, int n, int L, float *g,
                                     const GradientStep &step, int64_t d, hipStream_t stream)
{
    return with_short(tables, nodes_of(n, L), [&](const auto &t) { return launch_tree_decode(G, M, t, stored, n, L, g, step, d, stream); });
}

int decode_groups(int64_t d)
{
    const int64_t chunks = d < 4 ? d : (d + 3) / 4, per = d < kDecodeLongColumns ? 256 : 1024;
    return static_cast<int>((chunks + per - 1) / per);
}

hipError_t launch_decode(const float *M, float *g, const DecTerms &terms, const GradientStep &step, int64_t d, hipStream_t stream)
{
    const int nq = static_cast<int>(d >= 4 ? (d + 3) / 4 : d), groups = decode_groups(d);
    if (d < 4) decode_kernel<1, 8, 1, false><<<groups, 256, 0, stream>>>(M, g, terms, step, d, nq);
    else if (d < kDecodeLongColumns) decode_kernel<4, 8, 1, false><<<groups, 256, 0, stream>>>(M, g, terms, step, d, nq);
    else decode_kernel<4, 1, 4, true><<<groups, 256, 0, stream>>>(M, g, terms, step, d, nq);
    return hipGetLastError();
}

// ---- yardstick: a plain streaming read ------------------------------------------------------------------------------------
// Every workgroup walks one contiguous part of the array, eight non-temporal 16-byte loads in flight per thread; nothing but the
// loads and one add per word.  What this reaches is the practical ceiling for traffic that really comes from HBM (measured on
// MI355X: 7.0 to 7.1 TB/s; 6.0 to 6.3 without the non-temporal hint, or with a grid-wide stride instead of contiguous parts).
__global__ void __launch_bounds__(256) stream_read_kernel(const f4a *__restrict__ src, size_t n16, float *__restrict__ sink)
{
    const size_t per = ((n16 + gridDim.x - 1) / gridDim.x + 2047) / 2048 * 2048;      // whole unrolled iterations: parts start on 32 KB
    const size_t begin = per * blockIdx.x < n16 ? per * blockIdx.x : n16, end = begin + per < n16 ? begin + per : n16;
    float s = 0.f;
    size_t i = begin + threadIdx.x;
    for (; i + 7 * 256 < end; i += 8 * 256) {
        f4a v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(src + i + u * 256);
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u].x + v[u].y + v[u].z + v[u].w;
    }
    for (; i < end; i += 256) {
        const f4a v = __builtin_nontemporal_load(src + i);
        s += v.x + v.y + v.z + v.w;
    }
    s = wave_sum<true>(s);
    __shared__ float part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) sink[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

hipError_t launch_stream_read(const void *src, size_t n16, float *sink, hipStream_t stream)
{
    stream_read_kernel<<<kStreamGroups, 256, 0, stream>>>(static_cast<const f4a *>(src), n16, sink);
    return hipGetLastError();
}

// ---- device memory owned by the library --------------------------------------------------------------------------------
// For callers that cannot allocate (under stream capture, in serving loops): the scratch the aggregation needs beyond its inputs
// and outputs -- one encode program and the message rows M[N][d] -- lives in this array.  In host code the array's name is only a
// stand-in; its device address is asked for once per device, with that device current, and kept.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static __device__ __align__(256) unsigned char tables_of_trees[kTablePoolBytes];

namespace {
std::atomic<char *> g_scratch_ptr[kMaxDevices], g_tables_ptr[kMaxDevices];      // per device: where that device's copy of the array lives

hipError_t array_address(const void *name, std::atomic<char *> (&known)[kMaxDevices], char **ptr)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    char *p = known[dev].load(std::memory_order_acquire);
    if (!p) {
        void *sym = nullptr;
        e = hipGetSymbolAddress(&sym, name);
        if (e != hipSuccess) return e;
        if (!sym) return hipErrorInvalidSymbol;
        p = static_cast<char *>(sym);
        known[dev].store(p, std::memory_order_release);            // two threads racing here store the same address
    }
    *ptr = p;
    return hipSuccess;
}
}  // namespace

hipError_t static_scratch(char **ptr) { return array_address(HIP_SYMBOL(scratch), g_scratch_ptr, ptr); }
hipError_t table_pool(char **ptr) { return array_address(HIP_SYMBOL(tables_of_trees), g_tables_ptr, ptr); }

// Where the tree's tables do not fit the arguments of the launch that encodes (argument_tables), the encode program travels as kernel
// arguments of launches of its own (copied when the launch is enqueued) and one workgroup writes it out with vector stores.  What bounds
// it is the number of launches, 4 KB of arguments at most each, so a term of 28 bytes travels as 8: slab, row, level and the places of
// its two coefficients in a table of the block's distinct ones.  Every block is complete in itself, and only the terms that the mask
// leaves travel.  Ten vectors of 10 to 73728 entries on a tree of two levels of twelve with s = 2: 305 to
// 340 us with the program's bytes as they are (six launches per vector), 155 us in this form (one), 119 us with the tables as arguments.
struct ProgramBlock {
    static constexpr int kWords = 480;                   // 8-byte words: the coefficients, then the terms
    int32_t first, terms, coefs, subs;                   // subs: words of the sub-program table, behind the terms
    uint64_t word[kWords];
};
static_assert(sizeof(ProgramBlock) <= 4000, "kernel arguments");

__global__ void __launch_bounds__(256) program_kernel(ProgramTables out, ProgramBlock block)
{
    for (int i = threadIdx.x; i < block.terms; i += 256) {
        const uint64_t t = block.word[block.coefs + i];
        out.slab[block.first + i] = static_cast<int32_t>(t & 4095);
        out.row[block.first + i] = static_cast<int32_t>(t >> 12 & 4095) ^ -static_cast<int32_t>(t >> 52 & 1);      // ~row: not stored
        out.level[block.first + i] = static_cast<int32_t>(t >> 24 & 15);
        out.coef[block.first + i] = __longlong_as_double(static_cast<int64_t>(block.word[t >> 28 & 4095]));
        out.acoef[block.first + i] = __longlong_as_double(static_cast<int64_t>(block.word[t >> 40 & 4095]));
    }
    const int at = block.coefs + block.terms;
    for (int i = threadIdx.x; i < block.subs; i += 256) reinterpret_cast<uint64_t *>(out.sub)[i] = block.word[at + i];
}

hipError_t launch_program(const ProgramTables &out, const ProgramTables &host, int terms, int subs, hipStream_t stream)
{
    constexpr int kSlots = 2048;                         // of the hash table; a block has fewer than 480 distinct coefficients
    constexpr int kTailWords = 64;                       // groups have at most 64 members: their table leaves room for terms
    uint16_t slot[kSlots];
    ProgramBlock block;
    const int subs8 = subs / 2;
    static_assert(kTailWords < ProgramBlock::kWords, "the table fits a block");
    if (terms > 4096 || subs % 2 != 0 || subs8 > kTailWords) return hipErrorInvalidValue;
    bool tail = false;                                   // the sub-program table is on its way
    for (int first = 0; first < terms || !tail;) {
        std::memset(slot, 0xff, sizeof slot);
        int coefs = 0, count = 0;
        uint64_t packed[ProgramBlock::kWords];
        auto place = [&](double c) {                     // the coefficient's place in the block's table
            uint64_t bits;
            std::memcpy(&bits, &c, 8);
            unsigned h = static_cast<unsigned>((bits * 0x9E3779B97F4A7C15ull) >> 53);
            while (slot[h] != 0xffff && block.word[slot[h]] != bits) h = (h + 1) % kSlots;
            if (slot[h] == 0xffff) {
                slot[h] = static_cast<uint16_t>(coefs);
                block.word[coefs++] = bits;
            }
            return static_cast<uint64_t>(slot[h]);
        };
        while (first + count < terms && coefs + count + 3 <= ProgramBlock::kWords) {     // room for a term and two new coefficients
            const int t = first + count;
            const int32_t row = host.row[t] < 0 ? ~host.row[t] : host.row[t];
            if ((host.slab[t] | row) >> 12 || host.level[t] >> 4) return hipErrorInvalidValue;
            const uint64_t c = place(host.coef[t]), a = place(host.acoef[t]);
            packed[count++] = static_cast<uint64_t>(host.slab[t]) | static_cast<uint64_t>(row) << 12 | static_cast<uint64_t>(host.level[t]) << 24 |
                              c << 28 | a << 40 | static_cast<uint64_t>(host.row[t] < 0) << 52;
        }
        std::memcpy(block.word + coefs, packed, static_cast<size_t>(count) * 8);
        block.first = first;
        block.terms = count;
        block.coefs = coefs;
        block.subs = 0;
        first += count;
        const int used = coefs + count;
        if (first == terms && used + subs8 <= ProgramBlock::kWords) {
            block.subs = subs8;
            std::memcpy(block.word + used, host.sub, static_cast<size_t>(subs8) * 8);
            tail = true;
        }
        program_kernel<<<1, 256, 0, stream>>>(out, block);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---- the tables of a tree and a mask as one kernel argument --------------------------------------------------------------
namespace {
// the coefficient's place among the distinct ones, or -1: no room
int place_coefficient(double c, uint16_t *slot, uint64_t *value, int &values, int room)
{
    uint64_t bits;
    std::memcpy(&bits, &c, 8);
    unsigned h = static_cast<unsigned>((bits * 0x9E3779B97F4A7C15ull) >> 54);
    static_assert(TreeArguments::kSlots == 1 << 10 && TreeArguments::kSlots > 2 * ArgumentTables::kWords, "ten bits of hash, a table half empty");
    while (slot[h] != 0xffff && value[slot[h]] != bits) h = (h + 1) % TreeArguments::kSlots;
    if (slot[h] == 0xffff) {
        if (values == room) return -1;
        slot[h] = static_cast<uint16_t>(values);
        value[values++] = bits;
    }
    return slot[h];
}

int room_for_values(int halves) { return ArgumentTables::kWords - (halves + 3) / 4; }
}  // namespace

void lay_out_tree(int nodes, int slabs, const int32_t *node_begin, const double *slab_coef, TreeArguments *out)
{
    out->fits = false;
    out->nodes = nodes;
    out->values = 0;
    if (nodes > NodeCoefs::kNodes || slabs > 4 * ArgumentTables::kWords) return;
    out->halves = (nodes + 1) + nodes + slabs;
    const int room = room_for_values(out->halves);
    if (room <= 0) return;
    std::memset(out->slot, 0xff, sizeof out->slot);
    for (int i = 0; i <= nodes; ++i) out->half[i] = static_cast<uint16_t>(node_begin[i]);
    for (int i = 0; i < slabs; ++i) {
        const int k = place_coefficient(slab_coef[i], out->slot, out->value, out->values, room);
        if (k < 0) return;
        out->half[2 * nodes + 1 + i] = static_cast<uint16_t>(k);
    }
    out->fits = true;
}

bool argument_tables(const TreeArguments &tree, const NodeCoefs &coefs, ArgumentTables *out)
{
    if (!tree.fits) return false;
    const int room = room_for_values(tree.halves);
    uint16_t slot[TreeArguments::kSlots], places[NodeCoefs::kNodes];
    std::memcpy(slot, tree.slot, sizeof slot);
    std::memcpy(out->word, tree.value, static_cast<size_t>(tree.values) * 8);
    int values = tree.values;
    for (int i = 0; i < tree.nodes; ++i) {
        const int k = place_coefficient(coefs.a[i], slot, out->word, values, room);
        if (k < 0) return false;
        places[i] = static_cast<uint16_t>(k);
    }
    char *halves = reinterpret_cast<char *>(out->word + values);
    std::memcpy(halves, tree.half, static_cast<size_t>(tree.halves) * 2);
    std::memcpy(halves + (tree.nodes + 1) * 2, places, static_cast<size_t>(tree.nodes) * 2);
    out->at_begin = 4 * values;
    out->at_coef = out->at_begin + tree.nodes + 1;
    out->at_slab = out->at_coef + tree.nodes;
    out->used = values + (tree.halves + 3) / 4;
    return true;
}

// ---- where do workgroups run? -----------------------------------------------------------------------------------------
// __smid() packs the hardware ids of the wave: die (XCC) above 6 bits of shader engine and compute unit.
__global__ void __launch_bounds__(64) placement_probe_kernel(uint32_t *__restrict__ out)
{
    const unsigned id = __smid();
    if (threadIdx.x == 0) out[blockIdx.x] = ((id >> 6) << 16) | (id & 63u);
}

hipError_t launch_placement_probe(uint32_t *out, int groups, hipStream_t stream)
{
    placement_probe_kernel<<<groups, 64, 0, stream>>>(out);
    return hipGetLastError();
}

hipError_t launch_update(float *w, const float *g, float lr, int64_t d, hipStream_t stream)
{
    update_kernel<<<static_cast<unsigned>((d + 255) / 256), 256, 0, stream>>>(w, g, lr, d);
    return hipGetLastError();
}

hipError_t launch_measures(const double *sums, int64_t step_stride, int groups, int steps, bool with_star, float *metrics, hipStream_t stream)
{
    measures_kernel<<<steps, 256, 0, stream>>>(sums, step_stride, groups, with_star, metrics);
    return hipGetLastError();
}

}  // namespace cr
