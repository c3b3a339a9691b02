// Matrix-core kernel of libpconv for layers of few tiles (fp16 storage): the contraction of pconv_mfma.hip, cut so that
// a layer is over after few trips to memory rather than with the fewest bytes moved.
//
// What bounds such a layer is latency.  The kernel of pconv_mfma.hip takes a tile's channel blocks one after the other,
// and while the device is not full a block cannot take less than the round trip of the loads that fetch the next one
// (about 1.8 us): 16 blocks in sequence are 30 us, whatever the layer's size.  Here a workgroup's waves share a small
// tile -- AF*32 filters x BF*32 output pixels -- and each takes a part of the channel blocks, so the round trips of a
// tile's blocks run side by side; the partial sums meet in LDS at the end.
//
// A wave works alone until then: it stages its own blocks' activations in a part of the LDS that no other wave touches
// (no barriers), and takes its weights straight from memory into registers (no other wave of the workgroup wants them;
// waves of other workgroups find them in the L2).  While a block is multiplied, the next block's activations and each
// tap's weights are on their way into the registers that the current block has finished with.
//
// Tile: TH x TW output pixels of one image, chosen per layer (plan()); the staged patch is the (TH-1)*stride + 3 rows
// and (TW-1)*stride + 3 columns it reads, 16 channels deep, [half][row][column slot][8 channels].  Positions outside the
// image are loads outside the buffer descriptor, which return zero.
//
// Column slots.  A lane loads LW neighbouring columns at once (4, 2 or 1, whatever the row length allows), and its LW
// writes to LDS, one column each, would lie LW*16 bytes apart from its neighbour's: a 4-way bank conflict at LW = 4.  So
// the columns are dealt out by their residue modulo LW: column c lies in slot (c % LW) * Gp + c / LW.  Neighbouring lanes
// then write neighbouring slots; a tap is no longer a constant added to a pixel's slot, but depends on the tap's column
// only through three values per pixel; and at stride 2, where pixels take every other column, reads are free of
// conflicts too.  Gp is padded so that the residues' slots fall on different banks.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

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

struct SmallParams {
    const unsigned char* x;
    _Float16* y;
    const float* bias;
    const unsigned char* wq;    // MfmaWeights of tile height 64
    const unsigned* clist;      // as in MfmaParams
    const unsigned* tinfo;
    int N, C, F, H, W, Ho, Wo, stride, pad, relu;
    int CB, nt;                 // channel blocks of 16; tap slots
    int steps;                  // channel blocks a wave stages at a time, see the kernel: ceil(CB / NB)
    int row_off[9];             // per tap: bytes to its row of the patch, and its column
    int col[9];
    int TH, TW;                 // output pixels of a tile
    int tiles_m, tiles_x, tiles_y, tiles;
    int rs, cs;                 // image rows and columns between staged ones: 1, or the stride where no tap reads between them
    int PW;                     // columns per staged row
    int G;                      // pieces per staged row: PW / LW
    int Gp;                     // slots between the columns of one residue and the next's, see the kernel; G or more
    int row_bytes;              // slots of a staged row * 16
    int lead;                   // staged columns in front of the first tap's, so that pieces are aligned
    int items;                  // pieces of half a channel block: staged rows * G
    int item_stride;            // lanes they take: a multiple of 64 where that costs no more loads
    int plane_bytes;            // staged rows * row_bytes
    int pitch;                  // floats between two rows of partial sums
    int pv;                     // pixels per store: 4, 2 or 1
    int bias_off;               // bytes: the tile's biases lie behind the patches and the partial sums
    unsigned chan_bytes, img_bytes, wq_bytes;
    FastDiv div_m, div_x, div_y, div_G, div_TW, div_items;
};

// LW: pixels per load of the activations (0: channel-minor tensors, one load is eight channels of a position).  KI:
// pieces per lane and step.  NT: taps (0: fewer than nine, as the layer says).  A step is one channel block, or four of a
// layer of one tap: a block of those is four MFMAs, and its few pieces would leave most lanes of its loads idle.
template <int AF, int BF, int NT, int LW, int KI>
__global__ __launch_bounds__(512, 2) void small_conv_kernel(const SmallParams p) {
    constexpr bool NHWC = LW == 0;
    constexpr int NB = NT == 1 ? 4 : 1, TAPS = NT == 1 ? NB : 9, PX = BF * 32;
    extern __shared__ __align__(16) unsigned char lds[];
    // workgroups of one XCD (consecutive ids go round the XCDs) get consecutive tiles: the filter tiles of one patch
    // share an L2.  gridDim.x is a multiple of 8.
    const unsigned T = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (T >= (unsigned)p.tiles) return;
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lk = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = blockDim.x >> 6;
    unsigned r = fastdiv(T, p.div_m);
    const int tm = (int)(T - r * (unsigned)p.tiles_m);
    unsigned q = fastdiv(r, p.div_x);
    const int ox0 = (int)(r - q * (unsigned)p.tiles_x) * p.TW;
    r = fastdiv(q, p.div_y);
    const int oy0 = (int)(q - r * (unsigned)p.tiles_y) * p.TH, n = (int)r;
    const int s = p.stride, sr = p.rs > 1 ? 1 : s, sc = p.cs > 1 ? 1 : s;     // staged rows, columns per output row, column

    const int f0 = tm * AF * 32, wtile = f0 >> 6;
    int blocks = p.CB, wb = wtile * p.CB, steps = p.steps;
    if (p.clist) {
        blocks = (int)__builtin_amdgcn_readfirstlane(p.tinfo[2 * wtile]);
        steps = (blocks + NB - 1) / NB;
        wb = (int)__builtin_amdgcn_readfirstlane(p.tinfo[2 * wtile + 1]);
    }
    const int b0 = wave * steps / waves, b1 = (wave + 1) * steps / waves;      // this wave's steps

    // (one bias per thread for the epilogue, on its way while the blocks are multiplied)
    float bias_value = 0.f;
    if (p.bias && tid < AF * 32 && f0 + tid < p.F) bias_value = p.bias[f0 + tid];

    // staging: where each of this lane's pieces comes from in a channel's plane (or, channel-minor, in the image), and
    // where it goes in the wave's patch
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.x + (size_t)n * p.img_bytes, p.img_bytes);
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wq, p.wq_bytes);
    unsigned char* const patch = lds + wave * 2 * NB * p.plane_bytes;
    const int iy0 = oy0 * s - p.pad, ix0 = ox0 * s - p.pad - p.lead;
    constexpr int PIECE = NHWC ? 1 : LW;
    uint32_t goff[KI];
    int loff[KI], half[KI];
#pragma unroll
    for (int i = 0; i < KI; ++i) {
        const unsigned at = (unsigned)(lane + i * 64);
        const unsigned h = fastdiv(at, p.div_items), it = at - h * (unsigned)p.item_stride;
        const unsigned row = fastdiv(it, p.div_G);
        const int g = (int)(it - row * (unsigned)p.G), col = g * PIECE;
        const int iy = iy0 + (int)row * p.rs, ix = ix0 + col * p.cs;
        goff[i] = kInvalid;
        loff[i] = -1;
        half[i] = (int)h;
        if (h < 2 * NB && it < (unsigned)p.items) {
            loff[i] = (int)h * p.plane_bytes + (int)row * p.row_bytes + g * 16;
            if (iy >= 0 && iy < p.H && ix >= 0 && ix < p.W)
                goff[i] = NHWC ? (uint32_t)((iy * p.W + ix) * p.C + (int)h * 8) * 2u
                               : (uint32_t)(iy * p.W + ix) * 2u + (p.clist ? 0u : h * 8u * p.chan_bytes);
        }
    }
    Piece<NHWC ? 1 : LW> st[NHWC ? 1 : KI][8];
    uint4v sv[NHWC ? KI : 1];
    // (a channel behind the last is behind the end of the image: its offset is outside the descriptor, the load gives
    // zero; plan() has checked that the offsets of a last step's missing channels do not wrap round)
    auto load_patch = [&](int b) {
        if constexpr (NHWC) {
#pragma unroll
            for (int i = 0; i < KI; ++i) {
                const bool there = b * (16 * NB) + half[i] * 8 < p.C;          // (C is a multiple of 8: whole pieces)
                sv[i] = __builtin_amdgcn_raw_buffer_load_b128(xr, (int)(there ? goff[i] + (uint32_t)b * (32u * NB) : kInvalid), 0, 0);
            }
        } else {
            // (one branch around all loads: with one around each load the compiler waits for every load before the next)
            if (NB == 1 && p.clist) {
                uint32_t o0[8], o1[8];
#pragma unroll
                for (int ch = 0; ch < 8; ++ch) {
                    const unsigned* ids = p.clist + (size_t)(wb + b) * 16 + ch;
                    const unsigned c0 = __builtin_amdgcn_readfirstlane(ids[0]), c1 = __builtin_amdgcn_readfirstlane(ids[8]);
                    o0[ch] = c0 < (unsigned)p.C ? c0 * p.chan_bytes : kInvalid;
                    o1[ch] = c1 < (unsigned)p.C ? c1 * p.chan_bytes : kInvalid;
                }
#pragma unroll
                for (int ch = 0; ch < 8; ++ch)
#pragma unroll
                    for (int i = 0; i < KI; ++i) {
                        const uint32_t o = half[i] ? o1[ch] : o0[ch];
                        st[i][ch].load(xr, ((goff[i] | o) & kInvalid) ? kInvalid : goff[i] + o, 0);
                    }
            } else if (NB > 1 && p.clist) {
                // (a lane's eight channels depend on the lane: from the list by vector loads)
#pragma unroll
                for (int i = 0; i < KI; ++i) {
                    const int at = b * (16 * NB) + half[i] * 8;              // in the tile's list, of blocks * 16
                    const bool there = loff[i] >= 0 && at < blocks * 16 && !(goff[i] & kInvalid);
                    uint4v id[2] = {};
                    if (there) {
                        const uint4v* src = reinterpret_cast<const uint4v*>(p.clist + (size_t)wb * 16 + at);
                        id[0] = src[0];
                        id[1] = src[1];
                    }
#pragma unroll
                    for (int ch = 0; ch < 8; ++ch) {
                        const unsigned c = id[ch >> 2][ch & 3];
                        st[i][ch].load(xr, there && c < (unsigned)p.C ? goff[i] + c * p.chan_bytes : kInvalid, 0);
                    }
                }
            } else {
                const uint32_t o = (uint32_t)(b * (16 * NB)) * p.chan_bytes;
#pragma unroll
                for (int ch = 0; ch < 8; ++ch)
#pragma unroll
                    for (int i = 0; i < KI; ++i) st[i][ch].load(xr, goff[i] + (o + (uint32_t)ch * p.chan_bytes), 0);
            }
        }
    };
    auto write_patch = [&] {
#pragma unroll
        for (int i = 0; i < KI; ++i) {
            if (loff[i] < 0) continue;
            unsigned char* const to = patch + loff[i];
            if constexpr (NHWC) {
                *reinterpret_cast<uint4v*>(to) = sv[i];
            } else {
#pragma unroll
                for (int px = 0; px < LW; ++px) {
                    uint4v v;
                    v.x = interleave(st[i][0].dword(px >> 1), st[i][1].dword(px >> 1), px & 1);
                    v.y = interleave(st[i][2].dword(px >> 1), st[i][3].dword(px >> 1), px & 1);
                    v.z = interleave(st[i][4].dword(px >> 1), st[i][5].dword(px >> 1), px & 1);
                    v.w = interleave(st[i][6].dword(px >> 1), st[i][7].dword(px >> 1), px & 1);
                    *reinterpret_cast<uint4v*>(to + px * p.Gp * 16) = v;
                }
            }
        }
    };
    // weights of one tap: 16 bytes per lane and 32 filters
    half8 a[TAPS][AF];
    const int a_lane = (lk * 64 + (f0 & 63) + li) * 16;
    auto load_a = [&](int b, int ts) {
        // (blocks behind the last: nothing is loaded)
        const int block = NB == 1 ? b : b * NB + ts;
        const int voff = NB == 1 || block < blocks ? a_lane : (int)kInvalid;
        const int soff = NB == 1 || block < blocks ? ((wb + block) * p.nt + (NB == 1 ? ts : 0)) * (2 * 64 * 16) : 0;
#pragma unroll
        for (int af = 0; af < AF; ++af)
            a[ts][af] = __builtin_bit_cast(half8, __builtin_amdgcn_raw_buffer_load_b128(wr, voff + af * 512, soff, 0));
    };
    // operand positions of this lane's pixels, per column of the kernel
    constexpr int EXT = NT == 1 ? 1 : 3;
    int boff[EXT][BF];
#pragma unroll
    for (int bf = 0; bf < BF; ++bf) {
        const unsigned px = (unsigned)(bf * 32 + li), py = fastdiv(px, p.div_TW), pc = px - py * (unsigned)p.TW;
        const bool ok = (int)py < p.TH;
#pragma unroll
        for (int kx = 0; kx < EXT; ++kx) {
            const int c = (ok ? (int)pc * sc : 0) + (NT == 1 ? p.col[0] : kx + p.lead);
            boff[kx][bf] = lk * p.plane_bytes + (ok ? (int)py * sr * p.row_bytes : 0) + ((c % PIECE) * p.Gp + c / PIECE) * 16;
        }
    }
    float16v acc[AF][BF];
#pragma unroll
    for (int af = 0; af < AF; ++af)
#pragma unroll
        for (int bf = 0; bf < BF; ++bf)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[af][bf][i] = 0.f;
    // Lanes read what other lanes of their wave have written to the patch, and write over what others have read.  The
    // hardware takes a wave's LDS accesses in program order, so nothing has to wait; this keeps the compiler to it.
    auto hand_over = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    auto multiply = [&](int b, auto more) {
        // (the next block's loads, if there is one, are issued as the registers they fill become free)
        write_patch();
        hand_over();
        if constexpr (decltype(more)::value) load_patch(b + 1);
        // (the operands of a tap are read from LDS while the tap before is multiplied)
        half8 fb[2][BF];
        auto read_b = [&](int ts) {
#pragma unroll
            for (int bf = 0; bf < BF; ++bf) {
                int off;
                if constexpr (NT == 9) off = boff[ts % 3][bf] + (ts / 3) * p.row_bytes;
                else if constexpr (NT == 1) off = boff[0][bf] + p.row_off[0] + ts * 2 * p.plane_bytes;
                else off = (p.col[ts] == 0 ? boff[0][bf] : p.col[ts] == 1 ? boff[1][bf] : boff[2][bf]) + p.row_off[ts];
                fb[ts & 1][bf] = *reinterpret_cast<const half8*>(patch + off);
            }
        };
        read_b(0);
#pragma unroll
        for (int ts = 0; ts < TAPS; ++ts) {
            if (NT == 0 && ts >= p.nt) continue;
            if (ts + 1 < TAPS && (NT != 0 || ts + 1 < p.nt)) read_b(ts + 1);
#pragma unroll
            for (int bf = 0; bf < BF; ++bf)
#pragma unroll
                for (int af = 0; af < AF; ++af)
                    acc[af][bf] = NHWC ? __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ts][af], fb[ts & 1][bf], acc[af][bf], 0, 0, 0)
                                       : __builtin_amdgcn_mfma_f32_32x32x16_f16(fb[ts & 1][bf], a[ts][af], acc[af][bf], 0, 0, 0);
            if constexpr (decltype(more)::value) load_a(b + 1, ts);
        }
        if constexpr (decltype(more)::value) hand_over();
    };
    if (b0 < b1) {
        load_patch(b0);
#pragma unroll
        for (int ts = 0; ts < TAPS; ++ts)
            if (NT != 0 || ts < p.nt) load_a(b0, ts);
        int b = b0;
        for (; b + 1 < b1; ++b) multiply(b, std::true_type{});
        multiply(b, std::false_type{});
    }

    // ---- the waves' partial sums, 32 filters at a time, added in the order of the waves; bias, ReLU, store.
    // Channel-major (rows of the result are pixels, a lane's column its filter): [wave][filter][pixel], a thread adds and
    // stores pixels of a filter next to its neighbours; channel-minor (the other way round): [wave][pixel][filter].  Either
    // way a lane writes runs of four.
    // A workgroup comes here once, and what it runs comes from memory with it: channel-major, this is one loop over the
    // filters, not two copies, and its inner loop is not unrolled (channel-minor it is shorter, and lost by that: 128 -> 256 at
    // 14 x 14, batch 32, 9.6 -> 10.6 us).  (3,300 instructions for each 32 filters before, of which a workgroup ran
    // 200 in a dozen places: 3,500 to 4,300 clocks for the first 32 filters and 2,000 to 2,400 for the next, of 17,000 to
    // 34,000 in all.)
    float* const parts = reinterpret_cast<float*>(lds);
    float* const bias = reinterpret_cast<float*>(lds + p.bias_off);
    const int pitch = p.pitch, part = (NHWC ? PX : 32) * pitch;
    if (tid < AF * 32) bias[tid] = bias_value;               // (behind everything the waves still read)
    auto rounded = [&](float u) {
        if (p.relu) u = u > 0.f ? u : (u != u ? u : 0.f);
        return (_Float16)u;
    };
    auto store = [&](auto wave_count, int af) {
        constexpr int WAVES = decltype(wave_count)::value;
        const int fbase = f0 + af * 32;
        const float* const b = bias + af * 32;
        if constexpr (NHWC) {
            // a thread: four filters of one pixel
            const int fq = (tid & 7) * 4;
            if (fbase + fq >= p.F) return;                       // (F is a multiple of 8)
#pragma unroll
            for (int k = 0; k < (PX + WAVES * 8 - 1) / (WAVES * 8); ++k) {
                const int px = (tid >> 3) + k * WAVES * 8;
                const unsigned py = fastdiv((unsigned)px, p.div_TW);
                const int oy = oy0 + (int)py, ox = ox0 + px - (int)py * p.TW;
                if (px >= PX || (int)py >= p.TH || oy >= p.Ho || ox >= p.Wo) continue;
                float4v v[WAVES];
#pragma unroll
                for (int w = 0; w < WAVES; ++w) v[w] = *reinterpret_cast<const float4v*>(parts + w * part + px * pitch + fq);
                float4v sum = v[0];
#pragma unroll
                for (int w = 1; w < WAVES; ++w) sum += v[w];
                sum += *reinterpret_cast<const float4v*>(b + fq);
                _Float16 out[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) out[i] = rounded(sum[i]);
                uint2v o;
                __builtin_memcpy(&o, out, 8);
                *reinterpret_cast<uint2v*>(p.y + (((size_t)n * p.Ho + oy) * p.Wo + ox) * p.F + fbase + fq) = o;
            }
        } else {
            // a thread: PV neighbouring pixels of a row, as many as every tile's rows divide into (p.pv)
            auto rows = [&](auto vector_width) {
                constexpr int PV = decltype(vector_width)::value, QX = PX / PV, STEP = WAVES * 64 / QX;
                typedef float Vec __attribute__((ext_vector_type(PV)));
                const int px = (tid & (QX - 1)) * PV;
                const unsigned py = fastdiv((unsigned)px, p.div_TW);
                const int oy = oy0 + (int)py, ox = ox0 + px - (int)py * p.TW;
                if ((int)py >= p.TH || oy >= p.Ho || ox >= p.Wo) return;
                int f = tid / QX;
                const size_t step = (size_t)STEP * p.Ho * p.Wo;
                _Float16* y = p.y + (((size_t)n * p.F + fbase + f) * p.Ho + oy) * p.Wo + ox;
                const int most = min(32, p.F - fbase);
                const float* from = parts + f * pitch + px;
#pragma unroll 1
                for (; f < most; f += STEP, y += step, from += STEP * pitch) {
                    Vec v[WAVES];
#pragma unroll
                    for (int w = 0; w < WAVES; ++w) __builtin_memcpy(&v[w], __builtin_assume_aligned(from + w * part, sizeof(Vec)), sizeof(Vec));
                    Vec sum = v[0];
#pragma unroll
                    for (int w = 1; w < WAVES; ++w) sum += v[w];
                    sum += b[f];
                    _Float16 out[PV];
#pragma unroll
                    for (int i = 0; i < PV; ++i) out[i] = rounded(sum[i]);
                    __builtin_memcpy(__builtin_assume_aligned(y, 2 * PV), out, 2 * PV);
                }
            };
            if (p.pv == 4) rows(std::integral_constant<int, 4>{});
            else if (p.pv == 2) rows(std::integral_constant<int, 2>{});
            else rows(std::integral_constant<int, 1>{});
        }
    };
    auto put = [&](const float16v (&sums)[BF]) {
        float* const to = parts + wave * part + li * pitch + lk * 4;
#pragma unroll
        for (int bf = 0; bf < BF; ++bf)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                float4v v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = sums[bf][rq * 4 + i];
                *reinterpret_cast<float4v*>(to + (NHWC ? bf * 32 * pitch + rq * 8 : bf * 32 + rq * 8)) = v;
            }
    };
    if constexpr (NHWC) {
#pragma unroll
        for (int af = 0; af < AF; ++af) {
            __syncthreads();
            put(acc[af]);
            __syncthreads();
            if (waves == 8) store(std::integral_constant<int, 8>{}, af);
            else if (waves == 4) store(std::integral_constant<int, 4>{}, af);
            else if (waves == 2) store(std::integral_constant<int, 2>{}, af);
            else store(std::integral_constant<int, 1>{}, af);
        }
        return;
    }
    int halves = AF;
    asm volatile("" : "+s"(halves));                          // (one copy of the loop)
#pragma unroll 1
    for (int af = 0; af < halves; ++af) {
        __syncthreads();
        if (af == 0) put(acc[0]);
        else put(acc[AF - 1]);
        __syncthreads();
        if (waves == 8) store(std::integral_constant<int, 8>{}, af);
        else if (waves == 4) store(std::integral_constant<int, 4>{}, af);
        else if (waves == 2) store(std::integral_constant<int, 2>{}, af);
        else store(std::integral_constant<int, 1>{}, af);
    }
}

struct SmallShape {
    int af, bf;
};
const SmallShape kSmall[kSmallShapes] = {{1, 1}, {1, 2}, {2, 2}};

struct SmallPlan {
    SmallParams p;
    int lw, ki, waves;
    size_t lds;
    double us;               // estimated run time
};

// pieces per lane and step that the kernels are built for, by LW (0: channel-minor): the smallest of these that will do
const int kPieces[5][5] = {{1, 2, 3, 5, 9}, {1, 2, 3, 4, 0}, {1, 2, 3, 4, 0}, {}, {1, 2, 3, 0, 0}};
int pieces_for(int lw, long long need) {
    for (int k : kPieces[lw])
        if (k >= need) return k;
    return 0;
}

// The launch of one shape: tile, load width and waves with the smallest estimated time; false if the shape cannot take
// the layer in less than `bar` microseconds.
//
// The estimate (microseconds, fitted to ResNet-50's layers at batch 1 to 64 and some sixty ragged ones, inputs not in the
// L2): a workgroup takes a fixed time (first loads, the sums through LDS), up to twice as long when the compute unit is
// full, and a time per step of its waves: the round trip of the next step's loads, or what the load instructions of all
// waves on the compute unit take at one per 6 ns.  As many workgroups as registers and LDS allow share a compute unit, the
// rest waits for another round.  A full device is also bound by what its waves fetch from the L2, their weights above
// all: about 16 TB/s.
bool plan(const MfmaConv& a, int shape, double bar, SmallPlan* out) {
    const SmallShape& sh = kSmall[shape];
    const int M = sh.af * 32, PX = sh.bf * 32;
    if (a.groups > 1 || a.n_taps < 1 || a.n_taps > 9) return false;
    if (a.nhwc && (a.d_clist || a.C % 8 || a.F % 8)) return false;
    const int nb = a.n_taps == 1 ? 4 : 1;                    // channel blocks per step
    const unsigned long long img = (unsigned long long)a.C * a.H * a.W * 2ull;
    if ((unsigned long long)(a.C + 16 * nb) * a.H * a.W * 2ull >= 0x7FFFFFFFull) return false;
    const int ext = a.kext == 1 ? 1 : 3, s = a.stride;
    const uintptr_t xa = reinterpret_cast<uintptr_t>(a.x), ya = reinterpret_cast<uintptr_t>(a.y);
    const int tiles_m = (a.F + M - 1) / M;
    // (with channel lists: of a tile with the mean number of blocks)
    const int wtiles = (a.F + 63) / 64, blocks = a.d_clist ? (a.total_blocks + wtiles - 1) / wtiles : (a.C + 15) / 16;
    const int steps = (blocks + nb - 1) / nb;
    static const double kFixedUs[kSmallShapes] = {1.4, 2.2, 4.4}, kStepUs[kSmallShapes][2] = {{0.55, 0.35}, {0.8, 0.6}, {1.2, 0.9}};
    static const int kWavesPerCu[kSmallShapes][2] = {{16, 16}, {12, 16}, {8, 16}};
    // (a step of a 1x1 layer reads one short run from each of 64 planes: planes a multiple of 512 or of 2048 bytes apart
    // fall on few of the L2's channels, and the activations come at half or a quarter of the rate.  3,200 random layers,
    // 32 to 2048 channels: with the rate of other maps one in 140 was slower by a tenth or more than the tile kernel it
    // was chosen over -- 1082 -> 114 at 32 x 32, batch 11, 37.8 -> 54.4 us, where the 64 x 64 tile takes 24.6 -- so one in
    // 460.  Layers of nine taps, channel-minor tensors and stride 2 showed no such difference)
    const long long plane = 2ll * a.H * a.W;
    const double crowded = a.nhwc || ext != 1 || s != 1 || a.C < 64 ? 1.0 : plane % 2048 == 0 ? 4.0 : plane % 512 == 0 ? 2.0 : 1.0;
    SmallPlan best{};
    best.us = bar;
    bool found = false;
    const int cus = compute_units();
    const double out_us = (double)a.N * a.F * a.Ho * a.Wo * 2.0 / 4e6, step_weights = sh.af * 1024.0 * a.n_taps * nb;
    for (int tw = a.tile_w > 0 ? a.tile_w : std::min(PX, a.Wo); tw > 0; tw = a.tile_w > 0 ? 0 : tw - 1) {
        // (columns cut evenly, so that the last tile of a row is not nearly empty: the least width that makes as many tiles
        // of a row, then the next narrower one)
        const int nx = (a.Wo + tw - 1) / tw;
        tw = (a.Wo + nx - 1) / nx;
        int th = std::min(PX / tw, a.Ho);
        const int ny = (a.Ho + th - 1) / th;
        th = (a.Ho + ny - 1) / ny;
        const int rs = ext == 1 ? s : 1, rows = ext == 1 ? th : (th - 1) * s + ext;
        const long long tiles = (long long)tiles_m * nx * ny * a.N;
        if (tiles > 0x7FFFFFF0) continue;
        // (what no load width and no number of waves can make up for: a first call of a size pays for the search)
        const double busy_least = kFixedUs[shape] + (double)tiles * steps * kStepUs[shape][nb > 1] / ((double)cus * kWavesPerCu[shape][nb > 1]);
        if (3.0 + std::max(busy_least, (double)tiles * steps * step_weights / 16e6 + out_us) > best.us) continue;
        for (int lw = a.nhwc ? 0 : 4; lw >= 0; lw = lw == 4 ? 2 : lw == 2 ? 1 : -1) {
            if (a.tile_w > 0 && lw != a.tile_lw) continue;
            const int piece = lw ? lw : 1;
            if (lw > 1 && (a.W % lw || xa % (2 * lw) || (nx > 1 && tw * s % lw))) continue;
            const int lead = (piece - a.pad % piece) % piece;
            const int cs = ext == 1 && lw <= 1 ? s : 1;      // (loads of one column skip what a kernel of extent 1 does not read)
            const int pw = ext == 1 && lw <= 1 ? tw : ((tw - 1) * s + ext + lead + piece - 1) / piece * piece;
            const long long items = (long long)rows * (pw / piece);
            const int ki = pieces_for(lw, (items * 2 * nb + 63) / 64);
            if (!ki) continue;
            // (16 lanes read or write at a time, 256 bytes of banks: two residues' runs of 8 slots should lie 5 to 11
            // slots apart, four residues' runs of 4 slots 3 to 5 apart)
            int gp = pw / piece;
            if (lw == 2) while (gp % 16 < 5 || gp % 16 > 11) ++gp;
            if (lw == 4) while (gp % 8 < 3 || gp % 8 > 5) ++gp;
            const int row_slots = gp * piece;
            const int pitch = a.nhwc ? 36 : PX + 4;
            // a wave's step: bytes it fetches, and the instructions that take them
            // (a row of the patch comes in whole memory lines; the rows of a 1x1 layer are one run of pixels)
            const double row_bytes = ext == 1 && s == 1 ? pw * 2.0 : 64.0 + pw * cs * 2.0;
            const double fetched = step_weights + crowded * rows * row_bytes * 16.0 * nb;
            const int loads = (a.nhwc ? ki : 8 * ki) + sh.af * a.n_taps * nb;
            const double traffic_us = (double)tiles * steps * fetched / 16e6 + out_us;
            if (3.0 + std::max(busy_least, traffic_us) > best.us) continue;
            for (int waves = 8; waves >= 1; waves /= 2) {
                if (a.splits ? waves != a.splits : waves > steps && waves > 1) continue;
                const size_t stage = (size_t)rows * row_slots * 32 * nb * waves;
                const size_t parts = (size_t)waves * (a.nhwc ? PX : 32) * pitch * 4;
                const size_t bias_off = (std::max(stage, parts) + 15) / 16 * 16, lds = bias_off + M * 4;
                if (lds > 160 * 1024) continue;
                const long long resident = (long long)cus *
                                           std::max<long long>(1, std::min<long long>(kWavesPerCu[shape][nb > 1] / waves, (160 * 1024) / lds));
                const double per = (double)tiles / resident;
                const double rounds = per <= 1.0 ? 1.0 : per + 0.3 * (std::ceil(per) - per);
                const double on_cu = std::min((double)resident, std::max<double>(tiles, cus)) / cus * waves;
                const double busy = rounds * (kFixedUs[shape] * (1.0 + on_cu / 16.0) + 0.1 * waves +
                                              (steps + waves - 1) / waves * std::max(kStepUs[shape][nb > 1], on_cu * loads * 0.006));
                const double us = 3.0 + std::max(busy, traffic_us) + 0.15 * std::min(busy, traffic_us);
                // (of equal ones the narrowest tile, then the widest loads and the most waves)
                if (us > best.us || (us == best.us && (!found || best.p.TW == tw))) continue;
                best.us = us;
                found = true;
                SmallParams p{};
                p.TH = th; p.TW = tw; p.tiles_x = nx; p.tiles_y = ny; p.tiles = (int)tiles;
                p.rs = rs; p.cs = cs;
                p.PW = pw; p.lead = lead; p.items = (int)items;
                p.G = pw / piece; p.Gp = gp;
                p.row_bytes = row_slots * 16;
                p.plane_bytes = rows * p.row_bytes;
                p.pitch = pitch;
                p.bias_off = (int)bias_off;
                best.p = p;
                best.lw = lw; best.ki = ki; best.waves = waves; best.lds = lds;
            }
        }
    }
    if (!found) return false;
    SmallParams& p = best.p;
    p.x = static_cast<const unsigned char*>(a.x);
    p.y = static_cast<_Float16*>(a.y);
    p.bias = a.bias;
    p.wq = static_cast<const unsigned char*>(a.d_w);
    p.clist = a.d_clist;
    p.tinfo = a.d_tinfo;
    p.N = a.N; p.C = a.C; p.F = a.F; p.H = a.H; p.W = a.W; p.Ho = a.Ho; p.Wo = a.Wo;
    p.stride = s; p.pad = a.pad; p.relu = a.relu;
    p.CB = (a.C + 15) / 16;
    p.steps = (p.CB + nb - 1) / nb;
    p.nt = a.n_taps;
    for (int t = 0; t < p.nt; ++t) {
        p.row_off[t] = a.taps[t] / 3 * p.row_bytes;
        p.col[t] = a.taps[t] % 3 + (p.nt == 1 ? p.lead : 0);
    }
    p.pv = p.TW % 4 == 0 && a.Wo % 4 == 0 && ya % 8 == 0 ? 4 : p.TW % 2 == 0 && a.Wo % 2 == 0 && ya % 4 == 0 ? 2 : 1;
    p.tiles_m = tiles_m;
    p.chan_bytes = (unsigned)((size_t)a.H * a.W * 2);
    p.img_bytes = (unsigned)img;
    const size_t wq = a.d_clist ? a.w_bytes : mfma_weight_bytes(a.F, a.C, 64, a.n_taps);
    if (wq >= 0x7FFFFFFFull) return false;
    p.wq_bytes = (unsigned)wq;
    p.div_m = make_fastdiv((unsigned)p.tiles_m);
    p.div_x = make_fastdiv((unsigned)p.tiles_x);
    p.div_y = make_fastdiv((unsigned)p.tiles_y);
    p.div_G = make_fastdiv((unsigned)p.G);
    p.item_stride = p.items;
    if (((p.items + 63) / 64) * 2 * nb <= best.ki) p.item_stride = (p.items + 63) / 64 * 64;
    p.div_items = make_fastdiv((unsigned)p.item_stride);
    p.div_TW = make_fastdiv((unsigned)p.TW);
    *out = best;
    return true;
}

template <int AF, int BF>
int launch_shape(const SmallPlan& pl, hipStream_t st) {
    const int nt = pl.p.nt == 9 ? 9 : pl.p.nt == 1 ? 1 : 0;
    const dim3 grid((unsigned)((pl.p.tiles + 7) / 8 * 8)), block((unsigned)(pl.waves * 64));
#define PCONV_SMALL_CASE(LWv, KIv) PCONV_SMALL_ONE(9, LWv, KIv) PCONV_SMALL_ONE(1, LWv, KIv) PCONV_SMALL_ONE(0, LWv, KIv)
#define PCONV_SMALL_ONE(NTv, LWv, KIv)                                                                                 \
    if (nt == NTv && pl.lw == LWv && pl.ki == KIv) {                                                                   \
        auto kern = small_conv_kernel<AF, BF, NTv, LWv, KIv>;                                                          \
        static LdsAllowance allowed;                                                                                   \
        if (pl.lds > 64 * 1024) PCONV_HIP(allowed.ask((const void*)kern));                                             \
        hipLaunchKernelGGL(kern, grid, block, pl.lds, st, pl.p);                                                       \
        PCONV_HIP(hipGetLastError());                                                                                  \
        return PCONV_OK;                                                                                               \
    }
    PCONV_SMALL_CASE(1, 1) PCONV_SMALL_CASE(1, 2) PCONV_SMALL_CASE(1, 3) PCONV_SMALL_CASE(1, 4)
    PCONV_SMALL_CASE(2, 1) PCONV_SMALL_CASE(2, 2) PCONV_SMALL_CASE(2, 3) PCONV_SMALL_CASE(2, 4)
    PCONV_SMALL_CASE(4, 1) PCONV_SMALL_CASE(4, 2) PCONV_SMALL_CASE(4, 3)
    PCONV_SMALL_CASE(0, 1) PCONV_SMALL_CASE(0, 2) PCONV_SMALL_CASE(0, 3) PCONV_SMALL_CASE(0, 5) PCONV_SMALL_CASE(0, 9)
#undef PCONV_SMALL_CASE
#undef PCONV_SMALL_ONE
    return PCONV_EUNSUPPORTED;
}

}  // namespace

double small_estimate_us(MfmaConv* a, int shape, double bar) {
    SmallPlan pl;
    if (shape < 0 || shape >= kSmallShapes || !plan(*a, shape, bar, &pl)) return -1.0;
    a->tile_w = pl.p.TW;
    a->tile_lw = pl.lw;
    a->splits = pl.waves;
    return pl.us;
}

int launch_small_conv(const MfmaConv& a, int shape, void* stream) {
    SmallPlan pl;
    if (shape < 0 || shape >= kSmallShapes || !plan(a, shape, 1e30, &pl)) return PCONV_EUNSUPPORTED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    switch (shape) {
        case 0: return launch_shape<1, 1>(pl, st);
        case 1: return launch_shape<1, 2>(pl, st);
        default: return launch_shape<2, 2>(pl, st);
    }
}

}  // namespace pconv
