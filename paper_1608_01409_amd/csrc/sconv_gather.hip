// Gather kernels: small launches, straight from global memory.
//
// The LDS-tiled kernels pay a fixed price before the first multiply-add (a block has to be staged, 64 lanes have to
// find positions or images to work on, and a launch with few tiles splits its channels and adds the parts up in a
// second launch).  A call with little arithmetic never earns that back, so it runs here: no LDS staging, one launch,
// every operand read through the vector cache, the nonzeros of one output row shared by up to 8 waves (fully connected:
// 16).  The sums are kept in fp64: the waves wait for loads, not for the vector units, and a sum that is rounded once is as
// exact in any order as the chain of fp32 multiply-adds of the other kernels, also for rows of two or three nonzeros.  (The kernel with
// four positions per lane adds eight products in fp32 first; against 64 bits it is still closer than those chains.)
// Measured, per call with the host's part: 256 -> 384, 13x13, 3x3, batch 1: flat-stream kernel 15.7 us, a position per lane
// 9.4, four 7.0; fully connected 4096 -> 1000 at batch 4, density 0.25: 47 -> 5.7 us.
#include <hip/hip_runtime.h>

#include "sconv_device.h"

namespace sconv {

typedef float float4u __attribute__((ext_vector_type(4), aligned(4))); // activations need only 4-byte alignment
using const_u32 = const __attribute__((address_space(4))) unsigned;

__device__ float raw_buffer_load(int4v rsrc, int voffset, int soffset, int aux) __asm("llvm.amdgcn.raw.buffer.load.f32");

// Workgroup -> (tile of positions, group of rows).  Workgroup ids go round the 8 XCDs: tiles are taken 8 at a time, one per
// XCD, so that a tile's inputs come into one L2 only; the tiles left over are spread over all of them.
static __device__ __forceinline__ void tile_of_block(int n_tiles, int n_rowgroups, FastDiv d_rg, int &tile, int &rg)
{
    const int bid = blockIdx.x, whole = n_tiles & ~7, full = whole * n_rowgroups;
    if (bid < full) {
        const int slot = bid >> 3, q = fdiv(slot, d_rg);
        rg = slot - q * n_rowgroups;
        tile = q * 8 + (bid & 7);
    } else {
        const int q = fdiv(bid - full, d_rg);
        rg = bid - full - q * n_rowgroups;
        tile = whole + q;
    }
}

// ---------------------------------------------------------------- convolutions
//
// A wave owns one CSR row and T x 64 output positions, counted through the images (position p = image * OHW + y * OW
// + x), and walks its share of the row's nonzeros eight at a time.  A nonzero is two scalar words: the weight, and
// (byte offset of (c, r, s) << 3) | (31 - tap), tap = r * S + s; the byte offset is the scalar offset of a buffer
// load whose lane offset is the position, so a nonzero costs one load, one multiply-add and the two instructions
// that apply the zero padding: bit `tap` of the lane's mask says that this tap falls outside the image at the lane's
// position, and is moved into the lane offset's sign bit, beyond the buffer's end, where the load returns 0.  Bit 31
// is always set: padding entries (weight 0) use it.
struct GatherArgs {
    const unsigned *ent;
    const int *rowptr;       // in entries, multiples of 8
    const float *in;
    float *out;
    const float *bias;
    int relu;
    int K, OHW, OW, H, W, R, S, stride, pad;
    int in_img;              // floats per input image
    int P;                   // output positions of the call: N * OHW
    int shift_bytes;         // (pad * W + pad) * 4: lane offsets are relative to that many bytes before `in`
    int rec_bytes;           // bytes of the input + shift_bytes
    int n_tiles, n_rowgroups;    // workgroups along the positions, along K
    FastDiv d_rg, d_ohw, d_ow;
};

template <int T, int SPLIT>
__global__ void __launch_bounds__(SPLIT > 4 ? SPLIT * 64 : 256) sconv_gather_kernel(const GatherArgs a)
{
    constexpr int kRows = SPLIT >= 4 ? 1 : 4 / SPLIT;        // rows of a workgroup
    constexpr int U = SCONV_GATHER_CHUNK;
    __shared__ double part[SPLIT > 1 ? kRows * SPLIT * T * 64 : 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int tile, rg;
    tile_of_block(a.n_tiles, a.n_rowgroups, a.d_rg, tile, rg);
    const int row_l = wave / SPLIT, part_i = wave - row_l * SPLIT;
    const int k = rg * kRows + row_l;
    const bool live = k < a.K;
    const int p0 = tile * T * 64 + lane;

    unsigned base[T], inv[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int p = p0 + t * 64;
        const int n = fdiv(p, a.d_ohw), q = p - n * a.OHW;
        const int y = fdiv(q, a.d_ow), x = q - y * a.OW;
        const int iy = y * a.stride - a.pad, ix = x * a.stride - a.pad;
        unsigned cols = 0, m = 0;
        for (int s = 0; s < a.S; ++s) cols |= (ix + s >= 0 && ix + s < a.W) ? 0u : 1u << s;
        for (int r = 0; r < a.R; ++r) m |= ((iy + r >= 0 && iy + r < a.H) ? cols : (1u << a.S) - 1u) << (r * a.S);
        const bool out_of_range = p >= a.P;
        inv[t] = out_of_range ? 0xffffffffu : m | 0x80000000u;
        base[t] = out_of_range ? 0u : (unsigned)((n * a.in_img + (y * a.W + x) * a.stride) * 4);
    }
    double acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = 0.0;

    if (live) {
        const unsigned long long ip = (unsigned long long)a.in - (unsigned long long)a.shift_bytes;
        int4v rsrc;
        rsrc.x = __builtin_amdgcn_readfirstlane((int)(unsigned)ip);
        rsrc.y = __builtin_amdgcn_readfirstlane((int)(unsigned)(ip >> 32));
        rsrc.z = __builtin_amdgcn_readfirstlane(a.rec_bytes);
        rsrc.w = 0x00020000;
        const int j0 = ((const __attribute__((address_space(4))) int *)a.rowptr)[k];
        const int chunks = (((const __attribute__((address_space(4))) int *)a.rowptr)[k + 1] - j0) / U;
        const int mine = (chunks + SPLIT - 1) / SPLIT;
        const int c1 = min(chunks, (part_i + 1) * mine);
        const int c0 = part_i * mine;
        const_u32 *e = (const_u32 *)a.ent + 2 * ((size_t)j0 + (size_t)c0 * U);
        unsigned cur[2 * U], nxt[2 * U];
        if (c0 < c1) {
#pragma unroll
            for (int i = 0; i < 2 * U; ++i) cur[i] = e[i];
        }
        for (int c = c0; c < c1; ++c) {
            // the next chunk is requested before this one is used; the stream ends with a spare chunk
            e += 2 * U;
#pragma unroll
            for (int i = 0; i < 2 * U; ++i) nxt[i] = e[i];
            float v[U][T];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const unsigned ctl = cur[2 * u + 1];
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const unsigned off = ((inv[t] << (ctl & 31u)) & 0x80000000u) | base[t];
                    v[u][t] = raw_buffer_load(rsrc, (int)off, (int)(ctl >> 3 & ~3u), 0);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int t = 0; t < T; ++t) acc[t] = fma((double)__uint_as_float(cur[2 * u]), (double)v[u][t], acc[t]);
#pragma unroll
            for (int i = 0; i < 2 * U; ++i) cur[i] = nxt[i];
        }
    }
    if constexpr (SPLIT > 1) {
#pragma unroll
        for (int t = 0; t < T; ++t) part[((row_l * SPLIT + part_i) * T + t) * 64 + lane] = acc[t];
        __syncthreads();
        // the parts of a chunk are added by one wave, in order: chunk t by wave t % SPLIT of the row
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (t % SPLIT != part_i) continue;
            double v = 0.0;
#pragma unroll
            for (int i = 0; i < SPLIT; ++i) v += part[((row_l * SPLIT + i) * T + t) * 64 + lane];
            acc[t] = v;
        }
    }
    if (!live) return;
    const double b = a.bias ? (double)a.bias[k] : 0.0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        if (t % SPLIT != part_i) continue;
        const int p = p0 + t * 64;
        if (p >= a.P) continue;
        const int n = fdiv(p, a.d_ohw), q = p - n * a.OHW;
        float v = (float)(a.bias ? acc[t] + b : acc[t]);
        if (a.relu) v = fmaxf(v, 0.f);
        a.out[((size_t)n * a.K + k) * a.OHW + q] = v;
    }
}

template <int T, int SPLIT>
static int launch_gather_inst(const GatherArgs &a, int tiles, hipStream_t s, int *hip_err)
{
    hipLaunchKernelGGL((sconv_gather_kernel<T, SPLIT>), dim3((unsigned)(tiles * a.n_rowgroups)), dim3(SPLIT > 4 ? SPLIT * 64 : 256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        *hip_err = (int)e;
        return SCONV_ERR_HIP;
    }
    return SCONV_OK;
}

static int launch_gather4(const sconv_desc &d, const DeviceGather &dev, const GatherShape &gs, const float *in, float *out, int N,
                          const Epilogue &ep, void *stream, int *hip_err);

int launch_gather(const sconv_desc &d, const DeviceGather &dev, const GatherShape &gs, const float *in, float *out, int N,
                  const Epilogue &ep, void *stream, int *hip_err)
{
    const Geometry g = geometry(d);
    if (!gather_fits(d, N)) return SCONV_ERR_RANGE;
    if (gather4_fits(d)) return launch_gather4(d, dev, gs, in, out, N, ep, stream, hip_err);
    GatherArgs a;
    a.ent = static_cast<const unsigned *>(dev.ent);
    a.rowptr = static_cast<const int *>(dev.rowptr);
    a.in = in;
    a.out = out;
    a.bias = ep.bias;
    a.relu = ep.relu ? 1 : 0;
    a.K = d.K; a.OHW = g.OH * g.OW; a.OW = g.OW; a.H = d.H; a.W = d.W; a.R = d.R; a.S = d.S; a.stride = d.stride; a.pad = d.pad;
    a.in_img = d.C * d.H * d.W;
    a.P = N * a.OHW;
    a.shift_bytes = (d.pad * d.W + d.pad) * 4;
    a.rec_bytes = N * a.in_img * 4 + a.shift_bytes;
    const int rows = gs.split >= 4 ? 1 : 4 / gs.split;
    a.n_rowgroups = (d.K + rows - 1) / rows;
    const int tiles = (a.P + gs.t * 64 - 1) / (gs.t * 64);
    a.n_tiles = tiles;
    const int64_t grid = (int64_t)tiles * a.n_rowgroups;
    if (grid > 0x7fffffff) return SCONV_ERR_RANGE;
    a.d_rg = make_fastdiv(a.n_rowgroups, grid);
    const int64_t p_max = (int64_t)tiles * gs.t * 64;
    a.d_ohw = make_fastdiv(a.OHW, p_max);
    a.d_ow = make_fastdiv(a.OW, p_max);
    hipStream_t s = static_cast<hipStream_t>(stream);
#define X(TT, SP) if (gs.t == TT && gs.split == SP) return launch_gather_inst<TT, SP>(a, tiles, s, hip_err);
    X(1, 1) X(1, 2) X(1, 4) X(1, 8) X(2, 1) X(2, 2) X(2, 4) X(2, 8)
#undef X
    return SCONV_ERR_PLAN;
}

// The same with four neighbouring positions of an output row per lane, for stride 1.  A load instruction occupies the
// address unit for 16 clocks whether its lanes fetch 4 or 16 bytes (measured: 4.4 million multiply-adds per microsecond
// with a dword per lane, all of them in L1 or not), so a lane fetches 16.  The four words may leave the row: what a tap
// must not see is masked per word by the tap's bit of that position's mask.  They must not leave the tensor, so the
// nonzeros of its first and its last channel (the "edge" entries) take the dword loads above, word by word.
// Where an output row is as long as an input row, neighbours in the output stay neighbours in the input across the end of a row
// (what that brings into a window is masked like padding), and the fours may be counted through the whole image: 13x13 is 43 of them
// instead of 52.  They are where that leaves the fullest CU a workgroup less (gather4_flat; 14x14, 68 -> 96, batch 10, density 0.41: 11.6 ->
// 10.2 us).  A wave's head: a lane's four masks are runs of bits and a product (bit by bit they were most of it), and the stream's
// first chunk is on its way meanwhile: random layers of 4-20 us 1.00-1.11x, 1.03x on average (256 -> 384, 13x13, batch 1, 7.0 and 6.8 us,
// is within what its runs differ by).
struct Gather4Args {
    const unsigned *ent;     // like GatherArgs::ent, the low five bits being the tap itself
    const int *rows;         // per row: first entry, chunks of eight, edge entries behind them
    const float *in;
    float *out;
    const float *bias;
    int relu;
    int K, OHW, OW, H, W, R, S, pad;
    int in_img, Q, Q_img;    // fours of positions: of the call, of an image
    int flat;                // an output row is as long as an input row: fours are counted through the image, else through each row
    unsigned row_ones;       // bit r * S for every filter row
    int shift_bytes, rec_bytes, n_tiles, n_rowgroups;
    FastDiv d_rg, d_qimg, d_ow4, d_ow;
};

typedef float float4v __attribute__((ext_vector_type(4)));
__device__ float4v raw_buffer_load4(int4v rsrc, int voffset, int soffset, int aux) __asm("llvm.amdgcn.raw.buffer.load.v4f32");

template <int SPLIT>
__global__ void __launch_bounds__(SPLIT > 4 ? SPLIT * 64 : 256) sconv_gather4_kernel(const Gather4Args a)
{
    constexpr int kRows = SPLIT >= 4 ? 1 : 4 / SPLIT;
    constexpr int U = SCONV_GATHER_CHUNK;
    __shared__ double part[SPLIT > 1 ? kRows * SPLIT * 256 : 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int tile, rg;
    tile_of_block(a.n_tiles, a.n_rowgroups, a.d_rg, tile, rg);
    const int row_l = wave / SPLIT, part_i = wave - row_l * SPLIT;
    const int k = rg * kRows + row_l;
    const bool live = k < a.K;

    // the row's part of the stream, asked for before anything is computed
    const __attribute__((address_space(4))) int *row = (const __attribute__((address_space(4))) int *)a.rows + 3 * min(k, a.K - 1);
    const int j0 = row[0], chunks = row[1], edges = row[2];
    const int mine = (chunks + SPLIT - 1) / SPLIT;
    const int c0 = part_i * mine, c1 = min(chunks, c0 + mine);
    const_u32 *e = (const_u32 *)a.ent + 2 * ((size_t)j0 + (size_t)min(c0, chunks) * U), *ee = (const_u32 *)a.ent + 2 * ((size_t)j0 + (size_t)chunks * U);
    unsigned cur[2 * U], nxt[2 * U];
#pragma unroll
    for (int i = 0; i < 2 * U; ++i) cur[i] = e[i];            // (without a chunk: an edge entry, or what follows; the stream ends with a spare chunk)

    const int q = tile * 64 + lane;
    const int n = fdiv(q, a.d_qimg), rem = q - n * a.Q_img;
    const int y0 = a.flat ? 0 : fdiv(rem, a.d_ow4), x0 = a.flat ? rem * 4 : (rem - y0 * a.d_ow4.d) * 4;
    const int pos = y0 * a.OW + x0;                           // first of the four positions
    const bool on = q < a.Q;
    // Bit `tap`: this tap lies inside the image; bit 31 is clear.  The filter columns inside the image are a run of bits, repeated at every
    // filter row inside.
    auto rows_at = [&](int y) {
        const int r0 = min(max(a.pad - y, 0), a.R), r1 = min(max(a.H + a.pad - y, 0), a.R);
        return ((1u << r1 * a.S) - 1u) & ~((1u << r0 * a.S) - 1u) & a.row_ones;
    };
    auto cols_at = [&](int x) {
        const int s0 = min(max(a.pad - x, 0), a.S), s1 = min(max(a.W + a.pad - x, 0), a.S);
        return ((1u << s1) - 1u) & ~((1u << s0) - 1u);
    };
    unsigned valid[4];
    if (a.flat) {
        const int y = fdiv(x0, a.d_ow), x = x0 - y * a.OW;
        const unsigned rows0 = rows_at(y), rows1 = rows_at(y + 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool over = x + i >= a.OW;
            valid[i] = on && x0 + i < a.OHW ? cols_at(over ? x + i - a.OW : x + i) * (over ? rows1 : rows0) : 0u;
        }
    } else {
        const unsigned rows = rows_at(y0);
#pragma unroll
        for (int i = 0; i < 4; ++i) valid[i] = on && x0 + i < a.OW ? cols_at(x0 + i) * rows : 0u;
    }
    const unsigned base = on ? (unsigned)(n * a.in_img + (a.flat ? pos : y0 * a.W + x0)) * 4u : 0u;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};

    if (live) {
        const unsigned long long ip = (unsigned long long)a.in - (unsigned long long)a.shift_bytes;
        int4v rsrc;
        rsrc.x = __builtin_amdgcn_readfirstlane((int)(unsigned)ip);
        rsrc.y = __builtin_amdgcn_readfirstlane((int)(unsigned)(ip >> 32));
        rsrc.z = __builtin_amdgcn_readfirstlane(a.rec_bytes);
        rsrc.w = 0x00020000;
        for (int c = c0; c < c1; ++c) {
            e += 2 * U;                                       // the stream ends with a spare chunk
#pragma unroll
            for (int i = 0; i < 2 * U; ++i) nxt[i] = e[i];
            float4v v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = raw_buffer_load4(rsrc, (int)base, (int)(cur[2 * u + 1] >> 3 & ~3u), 0);
            __builtin_amdgcn_sched_barrier(0);                // all eight loads in flight
            // eight products in fp32, their sum to the fp64 one: the conversions are too slow for every product
            float s4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int m = __builtin_amdgcn_sbfe((int)valid[i], cur[2 * u + 1] & 31u, 1);
                    s4[i] = fmaf(__uint_as_float(cur[2 * u]), __uint_as_float(__float_as_uint(v[u][i]) & (unsigned)m), s4[i]);
                }
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i] += (double)s4[i];
#pragma unroll
            for (int i = 0; i < 2 * U; ++i) cur[i] = nxt[i];
        }
        // edge entries, shared by the waves of the row
        for (int j = part_i; j < edges; j += SPLIT) {
            const unsigned w = ee[2 * j], ctl = ee[2 * j + 1];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const unsigned off = (valid[i] >> (ctl & 31u) & 1u) ? base + 4u * i : 0x80000000u;
                acc[i] = fma((double)__uint_as_float(w), (double)raw_buffer_load(rsrc, (int)off, (int)(ctl >> 3 & ~3u), 0), acc[i]);
            }
        }
    }
    if constexpr (SPLIT > 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) part[((row_l * SPLIT + part_i) * 4 + i) * 64 + lane] = acc[i];
        __syncthreads();
        if (part_i != 0) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            double v = 0.0;
#pragma unroll
            for (int p = 0; p < SPLIT; ++p) v += part[((row_l * SPLIT + p) * 4 + i) * 64 + lane];
            acc[i] = v;
        }
    }
    if (!live || !on) return;
    const double b = a.bias ? (double)a.bias[k] : 0.0;
    float *dst = a.out + ((size_t)n * a.K + k) * a.OHW + pos;
    const int left = (a.flat ? a.OHW : a.OW) - x0;
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o[i] = (float)(a.bias ? acc[i] + b : acc[i]);
        if (a.relu) o[i] = fmaxf(o[i], 0.f);
    }
    if (left >= 4) {
        *(float4u *)dst = float4u{o[0], o[1], o[2], o[3]};
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < left) dst[i] = o[i];
    }
}

template <int SPLIT>
static int launch_gather4_inst(const Gather4Args &a, int tiles, hipStream_t s, int *hip_err)
{
    hipLaunchKernelGGL((sconv_gather4_kernel<SPLIT>), dim3((unsigned)(tiles * a.n_rowgroups)), dim3(SPLIT > 4 ? SPLIT * 64 : 256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        *hip_err = (int)e;
        return SCONV_ERR_HIP;
    }
    return SCONV_OK;
}

static int launch_gather4(const sconv_desc &d, const DeviceGather &dev, const GatherShape &gs, const float *in, float *out, int N,
                          const Epilogue &ep, void *stream, int *hip_err)
{
    const Geometry g = geometry(d);
    if (!gather4_fits(d)) return SCONV_ERR_PLAN;
    Gather4Args a;
    a.ent = static_cast<const unsigned *>(dev.ent);
    a.rows = static_cast<const int *>(dev.rowptr);
    a.in = in;
    a.out = out;
    a.bias = ep.bias;
    a.relu = ep.relu ? 1 : 0;
    a.K = d.K; a.OHW = g.OH * g.OW; a.OW = g.OW; a.H = d.H; a.W = d.W; a.R = d.R; a.S = d.S; a.pad = d.pad;
    a.in_img = d.C * d.H * d.W;
    const int ow4 = (g.OW + 3) / 4;
    a.flat = gather4_flat(d, N, gs.split);
    a.Q_img = a.flat ? (a.OHW + 3) / 4 : g.OH * ow4;
    a.row_ones = 0;
    for (int r = 0; r < d.R; ++r) a.row_ones |= 1u << r * d.S;
    a.Q = N * a.Q_img;
    a.shift_bytes = (d.pad * d.W + d.pad) * 4;
    a.rec_bytes = N * a.in_img * 4 + a.shift_bytes;
    const int rows = gs.split >= 4 ? 1 : 4 / gs.split;
    a.n_rowgroups = (d.K + rows - 1) / rows;
    const int tiles = (a.Q + 63) / 64;
    a.n_tiles = tiles;
    const int64_t grid = (int64_t)tiles * a.n_rowgroups;
    if (grid > 0x7fffffff) return SCONV_ERR_RANGE;
    a.d_rg = make_fastdiv(a.n_rowgroups, grid);
    a.d_qimg = make_fastdiv(a.Q_img, (int64_t)tiles * 64);
    a.d_ow4 = make_fastdiv(ow4, a.Q_img);
    a.d_ow = make_fastdiv(g.OW, a.OHW + 4);
    hipStream_t s = static_cast<hipStream_t>(stream);
#define X(SP) if (gs.split == SP) return launch_gather4_inst<SP>(a, tiles, s, hip_err);
    X(1) X(2) X(4) X(8)
#undef X
    return SCONV_ERR_PLAN;
}

// ---------------------------------------------------------------- fully connected layers, small batches
//
// out_t[k][n] = sum over the row's nonzeros of w * in_t[c][n].  The N images of a feature are contiguous, so a group
// of G = 2^LG >= N/4 lanes reads them as one run of 16-byte pieces and a wave works on 64 / G nonzeros at once, each
// lane group on its own; the groups' sums meet in a butterfly at the end, the SPLIT waves of a row in LDS.  With the
// flat-stream kernel the 64 lanes of a wave are positions of 4 images each: at a batch of 4 one lane of them works.
struct FcGatherArgs {
    const uint2 *ent;        // (weight, feature)
    const int *rowptr;
    const float *in_t;
    float *out_t;
    const float *bias;
    int relu;
    int K, N;
};

template <int LG, int SPLIT>
__global__ void __launch_bounds__(SPLIT > 4 ? SPLIT * 64 : 256) sconv_fc_gather_kernel(const FcGatherArgs a)
{
    constexpr int G = 1 << LG, kGroups = 64 >> LG;
    constexpr int kRows = SPLIT >= 4 ? 1 : 4 / SPLIT;
    constexpr int U = 4;
    __shared__ double4 part[SPLIT > 1 ? kRows * SPLIT * G : 1];
    const int lane = threadIdx.x & 63, grp = lane >> LG;
    const int q0 = lane & (G - 1), q = (int)blockIdx.y * G + q0;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int row_l = wave / SPLIT, part_i = wave - row_l * SPLIT;
    const int k = (int)blockIdx.x * kRows + row_l;
    const bool live = k < a.K;
    const int n4 = a.N >> 2;
    double4 acc = make_double4(0.0, 0.0, 0.0, 0.0);
    if (live) {
        const int r0 = a.rowptr[k], r1 = a.rowptr[k + 1];
        const int mine = ((r1 - r0 + SPLIT - 1) / SPLIT + kGroups - 1) / kGroups * kGroups;
        const int j0 = r0 + part_i * mine, j1 = min(r1, j0 + mine);
        const unsigned row_bytes = (unsigned)a.N * 4u;
        const unsigned q_bytes = (unsigned)min(q, n4 - 1) * 16u;  // lanes past the batch read its last piece and store nothing
        uint2 e[U], f[U];
        auto entries = [&](uint2 *to, int j) {                    // clamped: past the end the last entry again
#pragma unroll
            for (int u = 0; u < U; ++u) to[u] = a.ent[min(j + u * kGroups + grp, j1 - 1)];
        };
        if (j0 < j1) entries(e, j0);
        for (int j = j0; j < j1; j += U * kGroups) {
            float4u v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = *(const float4u *)((const char *)a.in_t + (e[u].y * row_bytes + q_bytes));
            entries(f, j + U * kGroups);                          // the next ones, requested before these are used
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // an entry past the end counts as 0 times 0, whatever its neighbour's activation is
                const bool on = j + u * kGroups + grp < j1;
                const double w = on ? (double)__uint_as_float(e[u].x) : 0.0;
                acc.x = fma(w, on ? (double)v[u].x : 0.0, acc.x);
                acc.y = fma(w, on ? (double)v[u].y : 0.0, acc.y);
                acc.z = fma(w, on ? (double)v[u].z : 0.0, acc.z);
                acc.w = fma(w, on ? (double)v[u].w : 0.0, acc.w);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) e[u] = f[u];
        }
    }
#pragma unroll
    for (int o = G; o < 64; o <<= 1) {
        acc.x += __shfl_xor(acc.x, o);
        acc.y += __shfl_xor(acc.y, o);
        acc.z += __shfl_xor(acc.z, o);
        acc.w += __shfl_xor(acc.w, o);
    }
    if constexpr (SPLIT > 1) {
        if (grp == 0) part[(row_l * SPLIT + part_i) * G + q0] = acc;
        __syncthreads();
        if (part_i != 0) return;
        acc = make_double4(0.0, 0.0, 0.0, 0.0);
#pragma unroll
        for (int i = 0; i < SPLIT; ++i) {
            const double4 p = part[(row_l * SPLIT + i) * G + q0];
            acc.x += p.x; acc.y += p.y; acc.z += p.z; acc.w += p.w;
        }
    }
    if (!live || grp != 0 || q >= n4) return;
    if (a.bias) {
        const double b = a.bias[k];
        acc.x += b; acc.y += b; acc.z += b; acc.w += b;
    }
    float4u o = {(float)acc.x, (float)acc.y, (float)acc.z, (float)acc.w};
    if (a.relu) {
        o.x = fmaxf(o.x, 0.f); o.y = fmaxf(o.y, 0.f); o.z = fmaxf(o.z, 0.f); o.w = fmaxf(o.w, 0.f);
    }
    *(float4u *)(a.out_t + (size_t)k * a.N + 4 * q) = o;
}

template <int LG, int SPLIT>
static int launch_fc_gather_inst(const FcGatherArgs &a, hipStream_t s, int *hip_err)
{
    constexpr int rows = SPLIT >= 4 ? 1 : 4 / SPLIT;
    hipLaunchKernelGGL((sconv_fc_gather_kernel<LG, SPLIT>), dim3((unsigned)((a.K + rows - 1) / rows), (unsigned)((a.N / 4 + (1 << LG) - 1) >> LG)),
                       dim3(SPLIT > 4 ? SPLIT * 64 : 256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        *hip_err = (int)e;
        return SCONV_ERR_HIP;
    }
    return SCONV_OK;
}

int launch_fc_gather(const sconv_desc &d, const DeviceGather &dev, const GatherShape &gs, const float *in_t, float *out_t, int N, const Epilogue &ep,
                     void *stream, int *hip_err)
{
    if (!fc_gather_fits(d, N)) return SCONV_ERR_RANGE;
    FcGatherArgs a;
    a.ent = static_cast<const uint2 *>(dev.ent);
    a.rowptr = static_cast<const int *>(dev.rowptr);
    a.in_t = in_t;
    a.out_t = out_t;
    a.bias = ep.bias;
    a.relu = ep.relu ? 1 : 0;
    a.K = d.K;
    a.N = N;
    hipStream_t s = static_cast<hipStream_t>(stream);
#define X(L) \
    if (gs.t == 1 << L) { \
        if (gs.split == 1) return launch_fc_gather_inst<L, 1>(a, s, hip_err); \
        if (gs.split == 4) return launch_fc_gather_inst<L, 4>(a, s, hip_err); \
        if (gs.split == 16) return launch_fc_gather_inst<L, 16>(a, s, hip_err); \
    }
    X(0) X(1) X(2) X(3) X(4) X(5)
#undef X
    return SCONV_ERR_PLAN;
}

} // namespace sconv
