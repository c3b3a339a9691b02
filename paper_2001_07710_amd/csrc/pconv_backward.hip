// Weight gradient of the pruned 3x3 layer for fp16 storage on gfx950 (MI355X): G[f][c][ky][kx] = sum over the batch's
// output pixels of dy[n][f][oy][ox] * x[n][c][oy+ky-1][ox+kx-1] (stride 1, padding 1), kept for the weights the layer
// keeps (the primal step of section 5.1 of the paper trains those by SGD through the masked layer: dL/dW = G o M).
//
// Why a dense contraction again.  Per tap this is a matrix product over the pixels, [filter][pixel] x [pixel][channel],
// and on this chip the fp16 matrix cores run it 16 times faster than the vector ALU would run the kept products
// alone; the mask is applied when the result is gathered.  Both operands are pixel-minor in NCHW, which is the K
// layout v_mfma_f32_32x32x16_f16 wants: a lane's operand is 8 consecutive pixels of one filter (or channel), 16
// contiguous bytes.  No transposition anywhere.
//
// Tile.  A workgroup owns 64 filters x 64 channels x 9 taps (four of its waves: 32 x 32 x 9 each, 144 accumulators)
// and walks over chunks of the pixels: R output rows x Gc groups of 8 columns of one image.  Per chunk it stages
//   x   [input row r'][group g][channel][8 pixels]            rows oy0-1 .. oy0+R, one 16-byte piece per (channel, r', g)
//   dy  [row r][group j][filter][8 pixels]                    groups one left and one right more than x has
// 1040 bytes from one (row, group) to the next, so that neighbouring groups of one channel fall on different banks
// when they are written and the 32 filters (channels) of an operand read lie side by side.  The three taps of a
// kernel row share one read of x: the sum over ox of dy[ox] * x[ox+kx-1] is the sum over x's own columns ox' of
// dy[ox'+1-kx] * x[ox'], so kx = 1 multiplies x with dy's group as it is, and kx = 0 / 2 with the same eight pixels of
// dy moved by one with the first / last pixel of the neighbouring group (eight v_alignbyte_b32 per K step of nine
// MFMAs).  Zero padding is nothing but dy's zero halo: columns beyond the image, rows beyond it, filters beyond F and
// channels beyond C are loads at an offset outside the buffer descriptor.
//
// Waves.  What bounded the first forms was that nothing overlapped: with one wave per SIMD that both stages and
// multiplies, the address arithmetic of 20 pieces, the wait for their loads, the LDS writes and two barriers added up
// with the MFMAs (matrix cores busy 29 % of the time).  So four waves, one per SIMD, do nothing but multiply, and four
// others, their neighbours on the SIMDs, nothing but stage: while chunk k is multiplied out of one half of the LDS they
// write chunk k + 1, whose loads were issued a chunk's time ago, into the other, and issue the loads of chunk k + 2.
// One barrier per chunk.  128 -> 128 channels at 112 x 112, batch 64: 341 -> 217 us, where the MFMAs alone, without
// loads and LDS reads, take 150 (the clock sinks to 1.95 GHz under them); 512 -> 512 at 28 x 28: 411 -> 258, at 14 x 14
// 179 -> 110.  256 -> 256 at 56 x 56: matrix cores busy 55 % of the time, LDS 38 % (a third of that bank conflicts).
//
// The pixels are split over S workgroups per tile; each writes its 9 x 64 x 64 partial sums to the workspace, a second
// kernel adds the S parts in order, 16 at a time, and a third adds those sums and gathers the sums of the kept weights into
// the canonical entry order of the packed layer (deterministic: no atomics).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "pconv_backward.h"
#include "pconv_internal.h"
#include "pconv_mfma_util.h"

namespace pconv {

#define PCONV_HIP(call)                                  \
    do {                                                 \
        hipError_t e_ = (call);                          \
        if (e_ != hipSuccess) {                          \
            pconv::set_hip_error(#call, (int)e_);        \
            return PCONV_EHIP;                           \
        }                                                \
    } while (0)

namespace {

constexpr int kPitch = 64 * 16 + 16;          // bytes from one (row, group) of a staged operand to the next
constexpr int kMaxSlots = 78;                 // (row, group) slots of a chunk, x and dy together: two chunks in 160 KB;
                                              // 64 / 256 of them 16-byte pieces per staging thread, 20 at most
constexpr int kTile = 64;

// Four neighbouring sums of the workspace.  The caller's pointer need be aligned no better than a float's, and the type says
// so; the compiler still moves 16 bytes at once, which the hardware does from any address.
typedef float sums4 __attribute__((ext_vector_type(4), aligned(4)));

struct GwParams {
    const unsigned char* x;
    const unsigned char* dy;
    float* ws;
    int N, C, F, H, W;
    int R, Gc, NJ;            // output rows and column groups per chunk; NJ = Gc + 2 staged groups of dy
    int nrb, ncb;             // row blocks and column blocks per image
    int chunks;               // N * nrb * ncb
    int S;                    // workgroups per tile
    int tiles_c, tiles;       // channel tiles; all tiles
    int slots_x, slots;       // (row, group) slots of a chunk: x's, and with dy's behind them
    unsigned x_img_bytes, dy_img_bytes;
    FastDiv div_Gc, div_NJ;
};

// eight consecutive fp16 elements from byte offset `off` (kInvalid: zeros), LW elements per load
template <int LW>
__device__ __forceinline__ uint4v load8(__amdgpu_buffer_rsrc_t r, const uint32_t (&off)[8 / LW]) {
    uint4v v;
    if constexpr (LW == 8) {
        v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off[0], 0, 0);
    } else if constexpr (LW == 4) {
        const uint2v a = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off[0], 0, 0);
        const uint2v b = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off[1], 0, 0);
        v = uint4v{a.x, a.y, b.x, b.y};
    } else if constexpr (LW == 2) {
        v.x = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off[0], 0, 0);
        v.y = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off[1], 0, 0);
        v.z = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off[2], 0, 0);
        v.w = __builtin_amdgcn_raw_buffer_load_b32(r, (int)off[3], 0, 0);
    } else {
        unsigned h[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) h[u] = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, (int)off[u], 0, 0);
        v = uint4v{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
    }
    return v;
}

// NP: pieces per staging thread and chunk, at most (8, 12, 16 or 20)
template <int LW, int NP>
__global__ __launch_bounds__(512, 2) void grad_weight_kernel(const GwParams p) {
    extern __shared__ __align__(16) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tile = (int)blockIdx.x / p.S, split = (int)blockIdx.x - tile * p.S;
    const int tf = tile / p.tiles_c, tc = tile - tf * p.tiles_c;
    const int R = p.R, Gc = p.Gc, NJ = p.NJ, H = p.H, W = p.W;
    const int buf_bytes = p.slots * kPitch;       // a staged chunk: x [r' < R + 2][g < Gc], then dy [r][j < NJ]
    // this workgroup's chunks: neighbours in the image, so that the rows two chunks share are still in the L2
    const int c0 = (int)((long long)split * p.chunks / p.S), c1 = (int)((long long)(split + 1) * p.chunks / p.S);

    if (wave >= 4) {
        // ---- staging.  This thread's pieces of a chunk (the same for every chunk): where they go in LDS, and where they
        // come from relative to the chunk's first output row and column.  A wave's 64 pieces are all of x or all of dy.
        // (Loads and LDS writes are unconditional -- a piece that is not there is a load outside the descriptor and a
        // write behind the two chunks -- because a branch around them makes the compiler wait for every load at once.)
        const int ltid = (int)threadIdx.x - 256, first = (wave - 4) * 64;
        int to[NP], rc[NP];                       // rc: relative row + 1 | (relative column + 8) << 16
        uint32_t rel[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int id = ltid + i * 256;
            const bool is_x = id < p.slots_x * 64;
            const int at = is_x ? id : id - p.slots_x * 64;
            const int groups = is_x ? Gc : NJ;
            const int q = (int)fastdiv((unsigned)at, is_x ? p.div_Gc : p.div_NJ), g = at - q * groups, c = q & 63, r = q >> 6;
            const int chan = (is_x ? tc : tf) * kTile + c;
            const int row = is_x ? r - 1 : r, col = is_x ? g * 8 : (g - 1) * 8;
            const bool there = id < p.slots * 64;
            to[i] = there ? ((is_x ? 0 : p.slots_x) + r * groups + g) * kPitch + c * 16 : 2 * buf_bytes + lane * 16;
            // (a piece that is not there, or of a filter or channel that is not: its loads lie outside the descriptor in every
            // chunk, at 2^31 and a pixel's place in one channel's image, which is below 2^31 as the whole image is)
            const bool read = there && chan < (is_x ? p.C : p.F);
            rel[i] = (read ? ((uint32_t)chan * (uint32_t)H + (uint32_t)row) * (uint32_t)W * 2u : kInvalid) + (uint32_t)(col * 2);
            rc[i] = (row + 1) | ((col + 8) << 16);
        }
        uint4v v[NP];
        // One chunk on: piece by piece, what has arrived is written into half `buf` and its register asks for the same piece
        // of the chunk after, so that every load has a whole chunk's time to come back.  (All writes first and then all
        // loads, the last loads' round trip was waited for in every chunk: 222 -> 217 us at 128 -> 128, 112 x 112.)
        auto move_on = [&](auto write_, auto load_, int buf, int chunk) {
            const int cb = chunk % p.ncb, q = chunk / p.ncb, rb = q % p.nrb, n = q / p.nrb;
            const int oy0 = rb * R - 1, col0 = cb * Gc * 8 - 8;                        // (matches rc's offsets)
            const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.x + (size_t)n * p.x_img_bytes, p.x_img_bytes);
            const __amdgpu_buffer_rsrc_t dr = make_rsrc(p.dy + (size_t)n * p.dy_img_bytes, p.dy_img_bytes);
            const int shift = (rb * R * W + cb * Gc * 8) * 2;
            // (which pieces are x's and which are there at all: asked anew for each chunk.  As conditions that do not
            // change the compiler would keep 2 NP of them, in more scalar registers than there are)
            int first_now = first;
            asm volatile("" : "+s"(first_now));
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if constexpr (decltype(write_)::value)
                    *reinterpret_cast<uint4v*>(lds + to[i] + (first_now + i * 256 < p.slots * 64 ? buf * buf_bytes : 0)) = v[i];
                if constexpr (decltype(load_)::value) {
                    const bool row_ok = (unsigned)(oy0 + (rc[i] & 0xFFFF)) < (unsigned)H;
                    const int col = col0 + (rc[i] >> 16);
                    uint32_t off[8 / LW];
#pragma unroll
                    for (int u = 0; u < 8 / LW; ++u)
                        off[u] = row_ok && (unsigned)(col + u * LW) < (unsigned)W ? rel[i] + (uint32_t)(shift + u * LW * 2)
                                                                                  : kInvalid;
                    v[i] = load8<LW>(first_now + i * 256 < p.slots_x * 64 ? xr : dr, off);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if (c0 >= c1) return;
        const std::true_type yes;
        const std::false_type no;
        move_on(no, yes, 0, c0);
        int chunk = c0;
        for (; chunk + 1 < c1; ++chunk) {
            move_on(yes, yes, (chunk - c0) & 1, chunk + 1);
            __syncthreads();
        }
        move_on(yes, no, (chunk - c0) & 1, 0);
        __syncthreads();
        __syncthreads();      // (the one in front of the last chunk's last step)
        return;
    }

    // ---- multiplying
    const int wf = wave >> 1, wc = wave & 1, li = lane & 31, lk = lane >> 5;
    float16v acc[3][3];
#pragma unroll
    for (int ky = 0; ky < 3; ++ky)
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[ky][kx][i] = 0.f;

    const int nk = R * Gc / 2;                  // K steps of 16 pixels per chunk (R*Gc is even)
    const int a_lane = p.slots_x * kPitch + (wf * 32 + li) * 16, b_lane = (wc * 32 + li) * 16;
    // This half-wave's items are lk, lk + 2, ...; item = r*Gc + g.  x has no halo groups, so an item's x slot is the
    // item number plus ky rows; its dy slot is r*NJ + g + 1, which skips the two halo groups at every row end.
    const bool one_group = Gc == 1;             // (then every item is a row of its own: three dy slots per item)
    const int a_off0 = (one_group ? lk * 3 + 1 : lk + 1) * kPitch + a_lane, b_off0 = lk * kPitch + b_lane;
    const int row_b = Gc * kPitch;
    if (c0 < c1) {
        // The K steps of all chunks are one sequence, software-pipelined: while a step's nine MFMAs run, the next step's
        // operands are read from LDS and shifted, a few instructions behind each MFMA, so that the wave never has more to
        // issue than an MFMA takes.  The barrier between two chunks stands in front of a chunk's last step, whose operands
        // are in registers by then: what it lets pass are the reads of the next chunk's first step.
        // The shifts by one pixel are made on the dy side: the sum over ox of dy[ox] * x[ox + kx - 1] is the sum over x's
        // own columns ox' of dy[ox' + 1 - kx] * x[ox'], so one read of x per kernel row serves its three taps, and dy is
        // read once per step and moved left and right by one pixel with its neighbour words (eight v_alignbyte_b32 per
        // nine MFMAs; with the shifts on the x side it was 24 vector instructions per step).
        const unsigned char *a_at = lds + a_off0, *b_at = lds + b_off0;
        uint4v cur;
        unsigned left, right;                   // the neighbouring groups' last and first two pixels
        auto read_a = [&] {
            cur = *reinterpret_cast<const uint4v*>(a_at);
            left = *reinterpret_cast<const unsigned*>(a_at - kPitch + 12);
            right = *reinterpret_cast<const unsigned*>(a_at + kPitch);
        };
        half8 a[2][3], b[3];                    // [kx]: dy at columns ox' + 1, ox', ox' - 1
        auto shift_a = [&](half8 (&to)[3]) {
            const unsigned l0 = __builtin_amdgcn_alignbyte(cur.x, left, 2);
            const unsigned l1 = __builtin_amdgcn_alignbyte(cur.y, cur.x, 2);
            const unsigned l2 = __builtin_amdgcn_alignbyte(cur.z, cur.y, 2);
            const unsigned l3 = __builtin_amdgcn_alignbyte(cur.w, cur.z, 2);
            const unsigned r3 = __builtin_amdgcn_alignbyte(right, cur.w, 2);
            to[2] = __builtin_bit_cast(half8, uint4v{l0, l1, l2, l3});
            to[1] = __builtin_bit_cast(half8, cur);
            to[0] = __builtin_bit_cast(half8, uint4v{l1, l2, l3, r3});
            asm volatile("" : "+v"(to[0]), "+v"(to[2]));       // (made here, not where the next step first needs them)
        };
        __builtin_amdgcn_s_setprio(1);
        __syncthreads();
        read_a();
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) b[ky] = *reinterpret_cast<const half8*>(b_at + ky * row_b);
        shift_a(a[0]);
        int g = lk, k = 0, buf = 0;
        auto step = [&](auto set_) {
            constexpr int set = decltype(set_)::value;
            g += 2;
            const bool wrap = g >= Gc;
            g = wrap ? g - Gc : g;
            a_at += (one_group ? 6 : wrap ? 4 : 2) * kPitch;
            b_at += 2 * kPitch;
            if (++k == nk) {
                __syncthreads();
                k = 0;
                g = lk;
                buf = buf_bytes - buf;
                a_at = lds + buf + a_off0;
                b_at = lds + buf + b_off0;
            }
            read_a();
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) {
                    __builtin_amdgcn_sched_barrier(0);
                    acc[ky][kx] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[set][kx], b[ky], acc[ky][kx], 0, 0, 0);
                }
                b[ky] = *reinterpret_cast<const half8*>(b_at + ky * row_b);
                if (ky == 1) shift_a(a[set ^ 1]);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        const long long steps = (long long)(c1 - c0) * nk;
        for (long long i = 0; i + 1 < steps; i += 2) {
            step(std::integral_constant<int, 0>{});
            step(std::integral_constant<int, 1>{});
        }
        if (steps & 1) step(std::integral_constant<int, 0>{});
    }

    // ---- partial sums: ws[split][tile][tap][wave][filter of the wave's 32][channel].  Accumulator row i of a 32 x 32 block
    // is filter (i/4)*8 + (lane/32)*4 + i%4, its column (lane%32) the channel; through a part of the LDS that no other
    // wave touches (all operands are in registers since the last barrier), so that every store is 1 KB in one piece.
    // (Straight from the registers, 128 bytes a row, the stores of a layer of a few chunks took as long as its MFMAs.)
    constexpr int kRow = 36;
    static_assert(4 * 32 * kRow * 4 <= 2 * 10 * kPitch, "a chunk has ten slots at least");
    float* const turn = reinterpret_cast<float*>(lds) + wave * 32 * kRow;
    sums4* const out = reinterpret_cast<sums4*>(p.ws + ((size_t)split * p.tiles + tile) * (9 * kTile * kTile));
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        // (lanes read what other lanes of the wave wrote; the hardware takes a wave's LDS accesses in order)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 16; ++i) turn[((i >> 2) * 8 + lk * 4 + (i & 3)) * kRow + li] = acc[t / 3][t % 3][i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < 4; ++q)
            out[((t * 4 + wave) * 4 + q) * 64 + lane] =
                *reinterpret_cast<const float4v*>(turn + (q * 8 + (lane >> 3)) * kRow + (lane & 7) * 4);
    }
}

// Where in a tile's part the sum of tap t for filter f and channel c of the tile lies
__device__ __forceinline__ int part_index(int t, int f, int c) {
    return ((t * 4 + (f >> 5) * 2 + (c >> 5)) * 32 + (f & 31)) * 32 + (c & 31);
}

// The S parts of every tile added up in groups of `cnt`, in order, each into its group's first part: a dense pass, four
// neighbouring sums per thread, so the parts are read at the rate of a copy.  (Summed inside the gather below instead, one scattered 4-byte read per part and kept
// weight, the parts of a layer with a single tile -- 256 of them -- took 90 us.)
__global__ __launch_bounds__(256) void grad_weight_reduce_kernel(float* __restrict__ ws, long long n4, long long part4, int S,
                                                                 int cnt) {
    // group blockIdx.y: parts group*cnt + s, s < cnt, as far as there are parts, added into the group's first
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    sums4* const w4 = reinterpret_cast<sums4*>(ws);
    const long long first = (long long)blockIdx.y * cnt;
    float4v sum = w4[first * part4 + i];
    for (int s = 1; s < cnt && first + s < S; ++s) sum += w4[(first + s) * part4 + i];
    w4[first * part4 + i] = sum;
}

// dw4[e][q] = sum over the parts that are left, in order, of the partial sum of entry e's filter and channel at the
// q-th tap of its pattern.  `stride`: floats from one of them to the next.
__global__ __launch_bounds__(256) void grad_weight_gather_kernel(const float* __restrict__ ws, const uint32_t* __restrict__ canon,
                                                                 float* __restrict__ dw4, long long n4, int parts,
                                                                 size_t stride, int tiles_c) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n4) return;
    const long long e = i >> 2;
    const int q = (int)(i & 3);
    const uint32_t f = canon[e * 2], cm = canon[e * 2 + 1], c = cm & 0xFFFFu, mask = cm >> 16;
    int t = -1, seen = 0;
    for (int b = 0; b < 9; ++b)
        if ((mask >> b) & 1u) {
            if (seen == q) t = b;
            ++seen;
        }
    float sum = 0.f;
    if (t >= 0) {
        const int tile = (int)(f / kTile) * tiles_c + (int)(c / kTile);
        const float* at = ws + (size_t)tile * (9 * kTile * kTile) + part_index(t, f % kTile, c % kTile);
        for (int s = 0; s < parts; ++s, at += stride) sum += *at;
    }
    dw4[i] = sum;
}

// Chunk geometry and the split of the pixels for a layer shape; false if the kernel cannot take it.
bool plan(const pconv_packed* p, int N, int H, int W, GwParams* out, int* lw, size_t* lds, size_t* ws_floats) {
    GwParams g{};
    g.N = N; g.C = p->C; g.F = p->F; g.H = H; g.W = W;
    const int Gp = (W + 7) / 8;
    g.ncb = (Gp + 7) / 8;
    g.Gc = (Gp + g.ncb - 1) / g.ncb;
    g.NJ = g.Gc + 2;
    // rows per chunk: as many as two chunks leave room for in LDS, evened out over the image; a K step is two items, so
    // rows x groups is even
    const int even = g.Gc % 2 ? 2 : 1;
    int R = (kMaxSlots - 2 * g.Gc) / (g.Gc + g.NJ) / even * even;
    int nrb = (H + R - 1) / R;
    R = ((H + nrb - 1) / nrb + even - 1) / even * even;
    nrb = (H + R - 1) / R;
    g.R = R;
    g.nrb = nrb;
    const long long chunks = (long long)N * nrb * g.ncb;
    if (chunks > 0x7FFFFFFF) return false;
    g.chunks = (int)chunks;
    g.tiles_c = (p->C + kTile - 1) / kTile;
    g.tiles = g.tiles_c * ((p->F + kTile - 1) / kTile);
    const int cus = compute_units();
    g.S = (int)std::max<long long>(1, std::min<long long>(chunks, (cus + g.tiles - 1) / g.tiles));
    g.div_Gc = make_fastdiv((unsigned)g.Gc);
    g.div_NJ = make_fastdiv((unsigned)g.NJ);
    g.slots_x = (R + 2) * g.Gc;
    g.slots = g.slots_x + R * g.NJ;
    const unsigned long long ximg = (unsigned long long)p->C * H * W * 2ull, dimg = (unsigned long long)p->F * H * W * 2ull;
    if (ximg >= 0x7FFFFFFFull || dimg >= 0x7FFFFFFFull) return false;
    g.x_img_bytes = (unsigned)ximg;
    g.dy_img_bytes = (unsigned)dimg;
    *lw = W % 8 == 0 ? 8 : W % 4 == 0 ? 4 : W % 2 == 0 ? 2 : 1;
    *lds = 2 * (size_t)g.slots * kPitch + 64 * 16;
    *ws_floats = (size_t)g.S * g.tiles * 9 * kTile * kTile;
    *out = g;
    return true;
}

int check_args(const pconv_packed* p, int N, int H, int W, int stride, int pad) {
    if (!p) return PCONV_EINVAL;
    if (N < 0 || H <= 0 || W <= 0) return PCONV_ESHAPE;
    if (p->dtype != PCONV_F16 || stride != 1 || pad != 1 || p->is_1x1) return PCONV_EUNSUPPORTED;
    for (uint16_t m : p->lib)
        if (__builtin_popcount(m) != 4) return PCONV_EUNSUPPORTED;      // (a derived form, not a layer from pconv_pack)
    return PCONV_OK;
}

}  // namespace
}  // namespace pconv

using namespace pconv;

extern "C" int pconv_conv3x3_grad_weight_workspace(const pconv_packed* p, int N, int H, int W, int stride, int pad,
                                                   size_t* bytes) {
    if (!bytes) return PCONV_EINVAL;
    *bytes = 0;
    if (int rc = check_args(p, N, H, W, stride, pad)) return rc;
    if (N == 0 || p->n_kept == 0) return PCONV_OK;
    GwParams g;
    int lw = 0;
    size_t lds = 0, floats = 0;
    if (!plan(p, N, H, W, &g, &lw, &lds, &floats)) return PCONV_EUNSUPPORTED;
    *bytes = floats * sizeof(float);
    return PCONV_OK;
}

extern "C" int pconv_conv3x3_grad_weight(const void* x, const void* dy, const pconv_packed* p, float* dw4, int N, int H,
                                         int W, int stride, int pad, void* workspace, size_t workspace_bytes,
                                         void* stream) {
    if (int rc = check_args(p, N, H, W, stride, pad)) return rc;
    if (!x || !dy || !dw4) return PCONV_EINVAL;
    if (!p->d_canon) return PCONV_ESTATE;
    int dev = -1;
    PCONV_HIP(hipGetDevice(&dev));
    if (dev != p->device) return PCONV_ESTATE;
    if (p->n_kept == 0) return PCONV_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const long long n4 = (long long)p->n_kept * 4;
    GwParams g;
    int lw = 0;
    size_t lds = 0, floats = 0;
    if (!plan(p, std::max(N, 1), H, W, &g, &lw, &lds, &floats)) return PCONV_EUNSUPPORTED;
    if (!workspace || workspace_bytes < floats * sizeof(float)) return PCONV_EINVAL;
    if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(dy)) % 2) return PCONV_EINVAL;
    // (the widest loads that the pointers allow as well as the row length)
    while (lw > 1 && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(dy)) % (2 * lw))) lw /= 2;
    g.x = static_cast<const unsigned char*>(x);
    g.dy = static_cast<const unsigned char*>(dy);
    g.ws = static_cast<float*>(workspace);
    g.N = N;
    if (N == 0) g.chunks = 0;          // (no pixels: the workgroups write zeros, the gather adds them)
    const dim3 grid((unsigned)(g.tiles * g.S));
    const int np = std::max(2, (g.slots + 15) / 16) * 4;         // (pieces: rounded up to what the kernel is built for)
#define PCONV_GW_CASE(LWv, NPv)                                                                                         \
    if (lw == LWv && np == NPv) {                                                                                       \
        auto kern = grad_weight_kernel<LWv, NPv>;                                                                       \
        static LdsAllowance allowed;                                                                                    \
        if (lds > 64 * 1024) PCONV_HIP(allowed.ask((const void*)kern));                                                 \
        hipLaunchKernelGGL(kern, grid, dim3(512), lds, st, g);                                                          \
    }
#define PCONV_GW_CASES(NPv) PCONV_GW_CASE(8, NPv) PCONV_GW_CASE(4, NPv) PCONV_GW_CASE(2, NPv) PCONV_GW_CASE(1, NPv)
    PCONV_GW_CASES(8) PCONV_GW_CASES(12) PCONV_GW_CASES(16) PCONV_GW_CASES(20)
#undef PCONV_GW_CASES
#undef PCONV_GW_CASE
    PCONV_HIP(hipGetLastError());
    // (groups of 16 consecutive parts, so that there are workgroups enough and the parts are read at the rate of a copy;
    // the groups' sums, 16 at most, the gather adds itself: a second such pass cost a launch, 4.5 us, and saved it 1)
    const int group = 16, groups = (g.S + group - 1) / group;
    const size_t part = (size_t)g.tiles * 9 * kTile * kTile;
    if (g.S > 1) {
        const long long part4 = (long long)(part / 4);
        hipLaunchKernelGGL(grad_weight_reduce_kernel, dim3((unsigned)((part4 + 255) / 256), (unsigned)groups), dim3(256), 0, st,
                           static_cast<float*>(workspace), part4, part4, g.S, group);
        PCONV_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(grad_weight_gather_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st,
                       static_cast<const float*>(workspace), p->d_canon, dw4, n4, groups, part * group, g.tiles_c);
    PCONV_HIP(hipGetLastError());
    return PCONV_OK;
}
