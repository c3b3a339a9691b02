// Host side of libpconv: argument checks, pattern assignment, connectivity selection, packing, export.
// Pure C++ (no HIP calls here); the device upload lives in pconv_device.hip.
#ifdef __SSE2__
#include <emmintrin.h>
#endif

#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <numeric>
#include <type_traits>

#include "pconv_internal.h"

namespace {

inline int popcount9(unsigned m) { return __builtin_popcount(m & 0x1FFu); }

// Library check shared by every entry point: K in [1,126], every mask a 9-bit value with exactly four bits
// (section 5.1 of the paper: four non-zero entries per kernel, at most C(9,4) = 126 masks).
int check_library(const uint16_t* lib, int K) {
    if (!lib) return PCONV_EINVAL;
    if (K < 1 || K > 126) return PCONV_EPATTERN;
    for (int j = 0; j < K; ++j)
        if (lib[j] >= 512u || popcount9(lib[j]) != 4) return PCONV_EPATTERN;
    return PCONV_OK;
}

// The library of a layer re-packed over parity planes: any masks with one to four bits.
int check_partial_library(const uint16_t* lib, int K) {
    if (!lib) return PCONV_EINVAL;
    if (K < 1 || K > 255) return PCONV_EPATTERN;
    for (int j = 0; j < K; ++j)
        if (lib[j] >= 512u || popcount9(lib[j]) < 1 || popcount9(lib[j]) > 4) return PCONV_EPATTERN;
    return PCONV_OK;
}

int check_fc(int F, int C) {
    if (F <= 0 || C <= 0 || C >= 65536) return PCONV_ESHAPE;
    if ((long long)F * (long long)C > (1ll << 31) / 9) return PCONV_ESHAPE;
    return PCONV_OK;
}

// Retained squared norm of one kernel under one mask: squares in double, added in ascending tap order.
inline double retained(const float* k9, unsigned m) {
    double acc = 0.0;
    bool first = true;
    for (int t = 0; t < 9; ++t) {
        if (!((m >> t) & 1u)) continue;
        const double v = (double)k9[t];
        const double sq = v * v;
        acc = first ? sq : acc + sq;
        first = false;
    }
    return acc;
}

}  // namespace

extern "C" int pconv_assign_patterns(const float* w, int F, int C, const uint16_t* lib, int K, uint8_t* pid_out) {
    if (!w || !pid_out) return PCONV_EINVAL;
    if (int rc = check_library(lib, K)) return rc;
    if (int rc = check_fc(F, C)) return rc;
    const long long n = (long long)F * C;
    for (long long i = 0; i < n; ++i) {
        const float* k9 = w + i * 9;
        int best = 0;
        double best_e = retained(k9, lib[0]);
        for (int j = 1; j < K; ++j) {
            const double e = retained(k9, lib[j]);
            if (e > best_e) {
                best_e = e;
                best = j;
            }
        }
        pid_out[i] = (uint8_t)best;
    }
    return PCONV_OK;
}

extern "C" int pconv_select_connectivity(const float* w, int F, int C, const uint16_t* lib, int K, const uint8_t* pid,
                                         double keep, uint8_t* mask_out) {
    if (!w || !pid || !mask_out) return PCONV_EINVAL;
    if (int rc = check_library(lib, K)) return rc;
    if (int rc = check_fc(F, C)) return rc;
    if (!(keep >= 0.0 && keep <= 1.0)) return PCONV_EINVAL;
    const long long n = (long long)F * C;
    for (long long i = 0; i < n; ++i)
        if (pid[i] >= K) return PCONV_EPATTERN;
    std::vector<double> score;
    std::vector<uint32_t> idx;
    try {
        score.resize((size_t)n);
        idx.resize((size_t)n);
    } catch (const std::bad_alloc&) {
        return PCONV_ENOMEM;
    }
    for (long long i = 0; i < n; ++i) score[(size_t)i] = retained(w + i * 9, lib[pid[i]]);
    std::iota(idx.begin(), idx.end(), 0u);
    long long k = (long long)std::floor(keep * (double)n + 0.5);
    k = std::max(0ll, std::min(k, n));
    auto before = [&](uint32_t a, uint32_t b) {
        if (score[a] != score[b]) return score[a] > score[b];
        return a < b;
    };
    if (k > 0 && k < n) std::nth_element(idx.begin(), idx.begin() + (k - 1), idx.end(), before);
    std::memset(mask_out, 0, (size_t)n);
    for (long long i = 0; i < k; ++i) mask_out[idx[(size_t)i]] = 1;
    return PCONV_OK;
}

namespace {

// The kept kernels of a layer, filter by filter with channels ascending: what every way of making a layer hands to
// pack_list.
struct KernelList {
    std::vector<uint32_t> row;        // [F+1]
    pconv::Array<uint16_t> c;         // channel
    pconv::Array<uint8_t> pid;        // pattern id
    pconv::Array<unsigned char> w4;   // the kept weights, taps ascending, four of the storage type (missing ones zero)
};

// Which of up to 64 mask bytes are set, as bits.  Where the host has no SSE2, eight bytes at a time in one word (256 x 256
// kernels: 3 us more of pconv_pack's 195 on the same machine).
inline uint64_t mask_bits(const uint8_t* m, int n) {
    uint8_t padded[64] = {};
    if (n < 64) m = static_cast<const uint8_t*>(std::memcpy(padded, m, (size_t)n));
    uint64_t removed = 0;
#ifdef __SSE2__
    for (int q = 0; q < 4; ++q) {
        const __m128i v = _mm_loadu_si128(reinterpret_cast<const __m128i*>(m + q * 16));
        removed |= (uint64_t)(unsigned)_mm_movemask_epi8(_mm_cmpeq_epi8(v, _mm_setzero_si128())) << (q * 16);
    }
#else
    for (int q = 0; q < 8; ++q) {
        uint64_t v = 0;
        for (int i = 0; i < 8; ++i) v |= (uint64_t)m[q * 8 + i] << (i * 8);
        // bit 7 of every byte that is zero, then the eight of them side by side in the top byte: byte i's goes there by
        // the factor's term 2^(49 - 7 i), and no two products of other terms meet in it
        v = ~(((v & 0x7F7F7F7F7F7F7F7Full) + 0x7F7F7F7F7F7F7F7Full) | v) & 0x8080808080808080ull;
        removed |= (v * 0x0002040810204081ull >> 56) << (q * 8);
    }
#endif
    return ~removed;
}

// From a dense tensor (of any alignment), pattern ids and a mask; false: the pattern id of a kept kernel is K or more.
// Kept and removed kernels follow no order that a branch predictor could learn, so the mask is read 64 kernels at a time
// and the loop goes from one set bit to the next.  (256 x 256 kernels, three tenths kept: 510 us for all of pconv_pack's
// host side with a branch or a byte per kernel and copies of lengths known at run time only, 190 now; 2.7 GHz.)
template <typename E>
bool list_kernels(const unsigned char* w, int F, int C, const uint16_t* lib, int K, const uint8_t* pid, const uint8_t* mask,
                  KernelList* out) {
    struct Taps {
        int at[4];
        E keep[4];                    // all ones, or zero where the pattern has fewer taps
    };
    std::vector<Taps> taps(256, Taps{});          // (any id can be looked up; those from K on are an error)
    for (int j = 0; j < K; ++j) {
        int q = 0;
        for (int t = 0; t < 9; ++t)
            if ((lib[j] >> t) & 1u) {
                taps[(size_t)j].at[q] = t;
                taps[(size_t)j].keep[q++] = (E)~(E)0;
            }
    }
    out->row.resize((size_t)F + 1);
    size_t n = 0;
    for (int f = 0; f < F; ++f) {
        const uint8_t* m = mask + (size_t)f * C;
        uint32_t kept = 0;
        for (int c = 0; c < C; ++c) kept += m[c] ? 1u : 0u;
        out->row[(size_t)f] = (uint32_t)n;
        n += kept;
    }
    out->row[(size_t)F] = (uint32_t)n;
    out->c.resize(n);
    out->pid.resize(n);
    out->w4.resize(n * 4 * sizeof(E));
    uint16_t* to_c = out->c.data();
    uint8_t* to_pid = out->pid.data();
    unsigned char* to_w4 = out->w4.data();
    bool bad = false;
    for (int f = 0; f < F; ++f)
        for (int c0 = 0; c0 < C; c0 += 64) {
            const size_t fc0 = (size_t)f * C + c0;
            for (uint64_t kept = mask_bits(mask + fc0, std::min(64, C - c0)); kept; kept &= kept - 1) {
                const int i = __builtin_ctzll(kept);
                const uint8_t j = pid[fc0 + i];
                bad |= j >= K;
                const Taps& t = taps[j];
                const unsigned char* k9 = w + (fc0 + i) * 9 * sizeof(E);
                E v[4];
                for (int q = 0; q < 4; ++q) {
                    std::memcpy(&v[q], k9 + (size_t)t.at[q] * sizeof(E), sizeof(E));
                    v[q] &= t.keep[q];
                }
                *to_c++ = (uint16_t)(c0 + i);
                *to_pid++ = j;
                std::memcpy(to_w4, v, sizeof(v));
                to_w4 += sizeof(v);
            }
        }
    return !bad;
}

// Finds the balanced order of `p` for the tiling that *out describes (see pconv::BalancedLayout).
void find_balanced(const pconv_packed* p, pconv::BalancedLayout* out) {
    const int F = p->F, C = p->C, K = p->K;
    const int fw = out->fw, fg = fw * out->nf, cc = out->cc;
    const int nch = out->n_chunks, npos = nch * cc;
    out->perm.assign((size_t)out->n_groups * npos, pconv::kNoChannel);
    out->pos_of.assign((size_t)out->n_groups * C, 0);

    // 16 chunks side by side in one vector of bytes: loads are at most nf * cc = 64
    constexpr int kMaxWaves = 16;
    constexpr uint8_t kFull = 192;                            // load of a chunk that takes no more channels
    typedef uint8_t Bytes __attribute__((vector_size(16)));
    const int nblk = (nch + 15) / 16;
    Bytes step[4];                                            // u in every byte, u <= nf <= 2
    for (int u = 0; u < 4; ++u)
        for (int i = 0; i < 16; ++i) step[u][i] = (uint8_t)u;
    std::vector<uint8_t> uses((size_t)C * kMaxWaves);        // [channel][wave] kept kernels of the wave's filters
    std::vector<uint32_t> weight((size_t)C), by_weight((size_t)fg + 2), order((size_t)C), fill((size_t)nch);
    std::vector<Bytes> load((size_t)nblk * kMaxWaves);        // [16 chunks][wave]
    std::vector<uint32_t> total((size_t)nblk * 16);           // per chunk: kernels << 12 | chunk
    std::vector<uint16_t> chunk_of((size_t)C);
    for (int g = 0; g < out->n_groups; ++g) {
        const int i0 = g * fg, i1 = std::min(F, i0 + fg);
        std::fill(uses.begin(), uses.end(), 0);
        std::fill(weight.begin(), weight.end(), 0u);
        for (int i = i0; i < i1; ++i) {
            const int w = (i - i0) % fw;                      // wave w holds positions i0 + w + a*fw
            const uint32_t e1 = p->grp_ptr[(size_t)(i + 1) * K];
            for (uint32_t e = p->grp_ptr[(size_t)i * K]; e < e1; ++e) {
                ++uses[(size_t)p->cin[e] * kMaxWaves + w];
                ++weight[p->cin[e]];
            }
        }
        // channels by decreasing number of users (at most fg; unused ones are dropped), then index: a counting sort
        std::fill(by_weight.begin(), by_weight.end(), 0u);
        for (int c = 0; c < C; ++c) ++by_weight[(size_t)fg - weight[(size_t)c] + 1];
        for (int u = 0; u <= fg; ++u) by_weight[(size_t)u + 1] += by_weight[(size_t)u];
        const uint32_t n_used = by_weight[(size_t)fg];
        for (int c = 0; c < C; ++c)
            if (weight[(size_t)c]) order[by_weight[(size_t)fg - weight[(size_t)c]]++] = (uint32_t)c;
        // greedy vector bin packing: put each channel into the chunk where the busiest wave stays least busy (then the
        // one with the fewest kernels, at most fg * cc = 1024, then the first of at most 4096: one number to minimise)
        std::fill(load.begin(), load.end(), step[0]);
        std::fill(fill.begin(), fill.end(), 0u);
        for (int k = 0; k < nblk * 16; ++k) total[(size_t)k] = (uint32_t)k;
        for (int k = nch; k < nblk * 16; ++k) load[(size_t)(k / 16) * kMaxWaves][k % 16] = kFull;
        for (uint32_t r = 0; r < n_used; ++r) {
            const uint32_t c = order[r];
            const uint8_t* u = &uses[(size_t)c * kMaxWaves];
            uint32_t best_key = ~0u;
            for (int blk = 0; blk < nblk; ++blk) {
                const Bytes* l = &load[(size_t)blk * kMaxWaves];
                Bytes mx = l[0] + step[u[0]];
                for (int w = 1; w < fw; ++w) {
                    const Bytes v = l[w] + step[u[w]];
                    mx = v > mx ? v : mx;
                }
                for (int k = 0; k < 16; ++k) {
                    const uint32_t key = total[(size_t)blk * 16 + k] + ((uint32_t)mx[k] << 23);
                    best_key = key < best_key ? key : best_key;
                }
            }
            const uint32_t best = best_key & 0xFFFu;
            Bytes* l = &load[(size_t)(best / 16) * kMaxWaves];
            for (int w = 0; w < fw; ++w) l[w][best % 16] = (uint8_t)(l[w][best % 16] + u[w]);
            total[best] += weight[c] << 12;
            if (++fill[best] == (uint32_t)cc) l[0][best % 16] = kFull;
            chunk_of[c] = (uint16_t)best;
        }
        // channels of a chunk in ascending order
        std::fill(fill.begin(), fill.end(), 0u);
        for (int c = 0; c < C; ++c) {
            if (!weight[(size_t)c]) continue;
            const uint32_t k = chunk_of[(size_t)c], pos = k * (uint32_t)cc + fill[k]++;
            out->pos_of[(size_t)g * C + c] = (uint16_t)pos;
            out->perm[(size_t)g * npos + pos] = (uint32_t)c;
        }
    }
}

// The tilings of the automatic choice (waves, filters per wave, channels per chunk; the 16-channel ones are the quad
// kernel's).
void plan_balanced(pconv_packed* p) {
    static const int tilings[5][3] = {{16, 2, 32}, {16, 1, 32}, {8, 1, 32}, {16, 2, 16}, {16, 1, 16}};
    p->balanced.resize(5);
    for (int t = 0; t < 5; ++t) {
        pconv::BalancedLayout& b = p->balanced[(size_t)t];
        b.fw = tilings[t][0];
        b.nf = tilings[t][1];
        b.cc = tilings[t][2];
        const int fg = b.fw * b.nf;
        b.n_groups = (p->F + fg - 1) / fg;
        b.n_chunks = (p->C + b.cc - 1) / b.cc;
        if (p->C > pconv::kOrderChannels) find_balanced(p, &b);
    }
}

// What the device needs to lay out the layer's weights in matrix-core order for workgroup tiles of mt filters (see
// pconv::MfmaWeights): tap slots and channel lists.
void plan_mfma_weights(const pconv_packed* p, int mt, int groups, pconv::MfmaWeights* out) {
    const int F = p->F, C = p->C, K = p->K;
    out->mt = mt;
    out->groups = groups;
    out->n_mtiles = (F + mt - 1) / mt;
    out->n_cblocks = (C / groups + 15) / 16;
    // taps that occur: the union of the masks of the patterns that have kept kernels
    unsigned present = 0;
    for (int i = 0; i < F; ++i)
        for (int j = 0; j < K; ++j)
            if (p->grp_ptr[(size_t)i * K + j + 1] > p->grp_ptr[(size_t)i * K + j]) present |= p->lib[(size_t)j];
    out->n_taps = 0;
    for (int t = 0; t < 9; ++t) {
        out->slot_of[t] = -1;
        if ((present >> t) & 1u) {
            out->slot_of[t] = (int8_t)out->n_taps;
            out->taps[out->n_taps++] = (uint8_t)t;
        }
    }
    // (channel ranges in the place of taps: as many tap slots as ranges, all of them the layer's one tap)
    if (groups > 1) {
        for (int g = 1; g < groups; ++g) out->taps[g] = out->taps[0];
        out->n_taps = groups;
    }
    // Channels that the filters of every tile keep.  Lists are made where they save at least a tenth of the blocks;
    // otherwise every tile takes all channels in their own order.
    // (A tile whose filters keep every channel between them, which unclustered connectivity comes to after a few of
    // them, looks at no more.)
    std::vector<uint8_t> used((size_t)out->n_mtiles * C, 0);
    std::vector<int> n_used((size_t)out->n_mtiles, 0);
    for (int i = 0; i < F; ++i) {
        const uint32_t t = p->filter_order[(size_t)i] / (uint32_t)mt;
        if (n_used[t] == C) continue;
        uint8_t* const u = &used[t * (size_t)C];
        int n = n_used[t];
        const uint32_t e1 = p->grp_ptr[(size_t)(i + 1) * K];
        for (uint32_t e = p->grp_ptr[(size_t)i * K]; e < e1; ++e) {
            n += 1 - u[p->cin[e]];
            u[p->cin[e]] = 1;
        }
        n_used[t] = n;
    }
    size_t listed = 0;
    for (int t = 0; t < out->n_mtiles; ++t) listed += std::max<size_t>(1, ((size_t)n_used[(size_t)t] + 15) / 16);
    const bool lists = groups == 1 && listed * 10 <= (size_t)out->n_mtiles * out->n_cblocks * 9;
    out->clist.clear();
    out->tinfo.clear();
    out->pos_of.clear();
    out->min_blocks = out->n_cblocks;
    out->total_blocks = out->n_mtiles * out->n_cblocks;
    if (lists) {
        out->min_blocks = 1 << 30;
        out->pos_of.assign((size_t)out->n_mtiles * C, 0);
        size_t at_block = 0;
        for (int t = 0; t < out->n_mtiles; ++t) {
            size_t n = 0;
            for (int c = 0; c < C; ++c)
                if (used[(size_t)t * C + c]) {
                    out->pos_of[(size_t)t * C + c] = (uint16_t)n++;
                    out->clist.push_back((uint32_t)c);
                }
            const size_t nb = std::max<size_t>(1, (n + 15) / 16);
            out->clist.resize((at_block + nb) * 16, pconv::kNoChannel);
            out->tinfo.push_back((uint32_t)nb);
            out->tinfo.push_back((uint32_t)at_block);
            out->min_blocks = std::min(out->min_blocks, (int)nb);
            at_block += nb;
        }
        out->total_blocks = (int)at_block;
    }
    out->elements = (size_t)out->total_blocks * out->n_taps * 2 * mt * 8;
}

// Packs a list of kept kernels: the canonical arrays, and what the device needs to make its layouts from them.  Masks
// of one to four taps, up to 255 of them; arguments are checked by the callers.
int pack_list(const KernelList& list, int dtype, int F, int C, const uint16_t* lib, int K, unsigned flags, bool want_mfma,
              bool one_by_one, pconv_packed** out) {
    const size_t kernel_bytes = dtype == PCONV_F16 ? 8 : 16;
    pconv_packed* p = new (std::nothrow) pconv_packed;
    if (!p) return PCONV_ENOMEM;
    try {
        p->F = F;
        p->C = C;
        p->K = K;
        p->dtype = dtype;
        p->lib.assign(lib, lib + K);
        const size_t n_kept = list.row[(size_t)F];
        p->n_kept = n_kept;

        // filter order: kept-kernel count descending, filter index ascending
        p->filter_order.resize((size_t)F);
        std::iota(p->filter_order.begin(), p->filter_order.end(), 0u);
        std::stable_sort(p->filter_order.begin(), p->filter_order.end(), [&](uint32_t a, uint32_t b) {
            return list.row[a + 1] - list.row[a] > list.row[b + 1] - list.row[b];
        });

        // canonical arrays: per (position i, pattern j) the kept kernels in ascending channel
        p->grp_ptr.assign((size_t)F * K + 1, 0);
        p->cin.resize(n_kept);
        p->w4.resize(n_kept * kernel_bytes);
        p->canon.resize(n_kept * 2);
        std::vector<uint32_t> at((size_t)K);
        uint32_t e = 0;
        for (int i = 0; i < F; ++i) {
            const uint32_t f = p->filter_order[(size_t)i], r0 = list.row[f], r1 = list.row[f + 1];
            std::fill(at.begin(), at.end(), 0u);
            for (uint32_t r = r0; r < r1; ++r) ++at[list.pid[r]];
            for (int j = 0; j < K; ++j) {
                const uint32_t n = at[(size_t)j];
                p->grp_ptr[(size_t)i * K + j] = at[(size_t)j] = e;
                e += n;
            }
            // (the bytes of a kernel's weights as a constant: a copy of a length that only the call knows is a call)
            auto place = [&](auto bytes) {
                constexpr size_t kBytes = decltype(bytes)::value;
                uint16_t* const cin = p->cin.data();
                uint32_t *const canon = p->canon.data(), *const next = at.data();
                unsigned char* const w4 = p->w4.data();
                for (uint32_t r = r0; r < r1; ++r) {
                    const uint32_t j = list.pid[r], d = next[j]++;
                    cin[d] = list.c[r];
                    canon[(size_t)d * 2] = f;
                    canon[(size_t)d * 2 + 1] = (uint32_t)list.c[r] | ((uint32_t)lib[j] << 16);
                    std::memcpy(w4 + d * kBytes, &list.w4[r * kBytes], kBytes);
                }
            };
            if (kernel_bytes == 8)
                place(std::integral_constant<size_t, 8>{});
            else
                place(std::integral_constant<size_t, 16>{});
        }
        p->grp_ptr[(size_t)F * K] = e;
        p->n_buckets = (C + pconv::kBucket - 1) / pconv::kBucket;

        plan_balanced(p);
        if (dtype == PCONV_F16 && want_mfma) {
            const int nh = (int)(sizeof(pconv::kMfmaTileHeights) / sizeof(int));
            p->mfma.resize((size_t)nh);
            for (int h = 0; h < nh; ++h) plan_mfma_weights(p, pconv::kMfmaTileHeights[h], 1, &p->mfma[(size_t)h]);
            // (a 1x1 layer is bound by the round trips of its many short channel blocks: kept a second time with
            // several channel ranges per block)
            if (one_by_one && K == 1 && C % (16 * pconv::kOneByOneGroups) == 0) {
                p->mfma.resize((size_t)(2 * nh));
                for (int h = 0; h < nh; ++h)
                    plan_mfma_weights(p, pconv::kMfmaTileHeights[h], pconv::kOneByOneGroups, &p->mfma[(size_t)(nh + h)]);
            }
        }
        const int rc = flags & PCONV_PACK_HOST_ONLY ? PCONV_OK : pconv::upload_packed(p);
        if (rc == PCONV_OK) {
            *out = p;
            return PCONV_OK;
        }
        pconv::release_device(p);
        delete p;
        return rc;
    } catch (const std::bad_alloc&) {
        pconv::release_device(p);
        delete p;
        return PCONV_ENOMEM;
    }
}

}  // namespace

// pconv_pack, and the packing of a layer re-packed over parity planes (`partial`: masks of one to four taps, up to
// 255 of them; missing taps of a kernel are stored as zero weights).
static int pack_impl(const void* w_oihw, int dtype, int F, int C, const uint16_t* lib, int K, const uint8_t* pid,
                     const uint8_t* mask, unsigned flags, bool partial, bool want_mfma, pconv_packed** out,
                     bool one_by_one = false) {
    if (!out) return PCONV_EINVAL;
    *out = nullptr;
    if (!w_oihw || !pid || !mask) return PCONV_EINVAL;
    if (dtype != PCONV_F32 && dtype != PCONV_F16) return PCONV_EINVAL;
    if (flags & ~(unsigned)PCONV_PACK_HOST_ONLY) return PCONV_EINVAL;
    if (int rc = partial ? check_partial_library(lib, K) : check_library(lib, K)) return rc;
    if (int rc = check_fc(F, C)) return rc;
    try {
        KernelList list;
        const unsigned char* wb = static_cast<const unsigned char*>(w_oihw);
        const bool ok = dtype == PCONV_F16 ? list_kernels<uint16_t>(wb, F, C, lib, K, pid, mask, &list)
                                           : list_kernels<uint32_t>(wb, F, C, lib, K, pid, mask, &list);
        if (!ok) return PCONV_EPATTERN;
        return pack_list(list, dtype, F, C, lib, K, flags, want_mfma, one_by_one, out);
    } catch (const std::bad_alloc&) {
        return PCONV_ENOMEM;
    }
}

extern "C" int pconv_pack(const void* w_oihw, int dtype, int F, int C, const uint16_t* lib, int K, const uint8_t* pid,
                          const uint8_t* mask, unsigned flags, pconv_packed** out) {
    return pack_impl(w_oihw, dtype, F, C, lib, K, pid, mask, flags, false, true, out);
}

// Bit t = 3*ky + kx of a mask moved to 3*(2-ky) + (2-kx) = 8 - t: the kernel rotated by 180 degrees.
static inline uint16_t rotate_mask(uint16_t m) {
    unsigned r = 0;
    for (int t = 0; t < 9; ++t)
        if ((m >> t) & 1u) r |= 1u << (8 - t);
    return (uint16_t)r;
}

extern "C" int pconv_packed_transpose(const pconv_packed* p, unsigned flags, pconv_packed** out) {
    if (!out) return PCONV_EINVAL;
    *out = nullptr;
    if (!p) return PCONV_EINVAL;
    if (flags & ~(unsigned)PCONV_PACK_HOST_ONLY) return PCONV_EINVAL;
    if (check_library(p->lib.data(), p->K) != PCONV_OK || p->is_1x1) return PCONV_EUNSUPPORTED;   // (a derived form)
    const int F = p->F, C = p->C, K = p->K;
    if (F >= 65536) return PCONV_ESHAPE;                 // (the filters become the input channels: 16-bit indices)
    const size_t esize = p->dtype == PCONV_F16 ? 2 : 4;
    try {
        std::vector<uint16_t> lib((size_t)K);
        for (int j = 0; j < K; ++j) lib[(size_t)j] = rotate_mask(p->lib[(size_t)j]);
        // the kernels by channel, filters ascending: filters are visited in that order and dropped into their channel's
        // row.  Tap t becomes tap 8 - t, so the kept weights of a kernel come in the opposite order.
        std::vector<uint32_t> pos_of_filter((size_t)F);
        for (int i = 0; i < F; ++i) pos_of_filter[p->filter_order[(size_t)i]] = (uint32_t)i;
        KernelList list;
        list.row.assign((size_t)C + 1, 0);
        for (size_t e = 0; e < p->n_kept; ++e) ++list.row[(size_t)p->cin[e] + 1];
        for (int c = 0; c < C; ++c) list.row[(size_t)c + 1] += list.row[(size_t)c];
        list.c.resize(p->n_kept);
        list.pid.resize(p->n_kept);
        list.w4.resize(p->n_kept * 4 * esize);
        std::vector<uint32_t> at(list.row.begin(), list.row.end() - 1);
        auto turn = [&](auto element) {
            typedef decltype(element) E;
            const E* const from = reinterpret_cast<const E*>(p->w4.data());
            E* const to = reinterpret_cast<E*>(list.w4.data());
            const uint16_t* const cin = p->cin.data();
            const uint32_t* const ptr = p->grp_ptr.data();
            uint16_t* const to_c = list.c.data();
            uint8_t* const to_pid = list.pid.data();
            uint32_t* const next = at.data();
            for (int f = 0; f < F; ++f) {
                const size_t i = pos_of_filter[(size_t)f];
                for (int j = 0; j < K; ++j)
                    for (uint32_t e = ptr[i * K + j], e1 = ptr[i * K + j + 1]; e < e1; ++e) {
                        const size_t d = next[cin[e]]++;
                        to_c[d] = (uint16_t)f;
                        to_pid[d] = (uint8_t)j;
                        for (int k = 0; k < 4; ++k) to[d * 4 + 3 - k] = from[(size_t)e * 4 + k];
                    }
            }
        };
        if (esize == 2)
            turn(uint16_t{});
        else
            turn(uint32_t{});
        return pack_list(list, p->dtype, C, F, lib.data(), K, flags, true, false, out);
    } catch (const std::bad_alloc&) {
        return PCONV_ENOMEM;
    }
}

extern "C" int pconv_pack_1x1(const void* w_fc, int dtype, int F, int C, const uint16_t* lib, int K, const uint8_t* pid,
                              const uint8_t* mask, unsigned flags, pconv_packed** out) {
    if (!out) return PCONV_EINVAL;
    *out = nullptr;
    if (!w_fc || !pid || !mask) return PCONV_EINVAL;
    if (dtype != PCONV_F32 && dtype != PCONV_F16) return PCONV_EINVAL;
    if (int rc = check_library(lib, K)) return rc;
    if (int rc = check_fc(F, C)) return rc;
    const int G = (C + 8) / 9;
    for (long long i = 0; i < (long long)F * G; ++i)
        if (mask[i] && pid[i] >= K) return PCONV_EPATTERN;
    const size_t esize = dtype == PCONV_F16 ? 2 : 4;
    const unsigned char* wb = static_cast<const unsigned char*>(w_fc);
    try {
        // the same layer as a 3x3 layer whose kernels keep their centre tap only: kernel (f,c) exists where channel c
        // is a kept position of its group's pattern
        std::vector<unsigned char> w9((size_t)F * C * 9 * esize, 0);
        std::vector<uint8_t> pid9((size_t)F * C, 0), mask9((size_t)F * C, 0);
        for (int f = 0; f < F; ++f)
            for (int c = 0; c < C; ++c) {
                const size_t fg = (size_t)f * G + (size_t)(c / 9);
                if (!mask[fg] || !((lib[pid[fg]] >> (c % 9)) & 1u)) continue;
                const size_t fc = (size_t)f * C + c;
                mask9[fc] = 1;
                std::memcpy(&w9[(fc * 9 + 4) * esize], wb + fc * esize, esize);
            }
        const uint16_t centre = 0x010;
        const int rc = pack_impl(w9.data(), dtype, F, C, &centre, 1, pid9.data(), mask9.data(), flags, true, true, out, true);
        if (rc == PCONV_OK) (*out)->is_1x1 = true;
        return rc;
    } catch (const std::bad_alloc&) {
        return PCONV_ENOMEM;
    }
}

int pconv::derive_for_stride2(const pconv_packed* p, int pad, bool upload, pconv_packed** out) {
    if (!p || !out || (pad != 0 && pad != 1)) return PCONV_EINVAL;
    *out = nullptr;
    const int F = p->F, C = p->C, K = p->K, C4 = 4 * C;
    if (C4 >= 65536) return PCONV_EUNSUPPORTED;
    const size_t esize = p->dtype == PCONV_F16 ? 2 : 4;
    try {
        // where tap t of a kernel goes: plane (0..3) and tap inside the plane's kernel
        int plane_of[9], tap_of[9];
        for (int t = 0; t < 9; ++t) {
            const int dy = t / 3 - pad, dx = t % 3 - pad;            // -1..2
            const int a = dy & 1, b = dx & 1;                          // parity (two's complement: -1 & 1 == 1)
            const int ky = (dy - a) / 2 + pad, kx = (dx - b) / 2 + pad;   // floor(d/2) + pad, in {0,1}
            plane_of[t] = 2 * a + b;
            tap_of[t] = 3 * ky + kx;
        }
        std::vector<unsigned char> w((size_t)F * C4 * 9 * esize, 0);
        std::vector<uint16_t> m9((size_t)F * C4, 0);
        for (int i = 0; i < F; ++i) {
            const uint32_t f = p->filter_order[(size_t)i];
            for (int j = 0; j < K; ++j) {
                int taps[4], q = 0;
                for (int t = 0; t < 9; ++t)
                    if ((p->lib[(size_t)j] >> t) & 1u) taps[q++] = t;
                for (uint32_t e = p->grp_ptr[(size_t)i * K + j]; e < p->grp_ptr[(size_t)i * K + j + 1]; ++e) {
                    const size_t c = p->cin[e];
                    for (int k = 0; k < q; ++k) {          // (q < 4: a layer whose kernels keep fewer taps, the 1x1 form)
                        const size_t fc = (size_t)f * C4 + 4 * c + (size_t)plane_of[taps[k]];
                        std::memcpy(&w[(fc * 9 + (size_t)tap_of[taps[k]]) * esize], &p->w4[((size_t)e * 4 + k) * esize], esize);
                        m9[fc] |= (uint16_t)(1u << tap_of[taps[k]]);
                    }
                }
            }
        }
        // library of the re-packed layer: the masks that occur, ascending
        std::vector<int> index_of(512, -1);
        std::vector<uint16_t> lib;
        std::vector<char> used(512, 0);
        for (size_t i = 0; i < m9.size(); ++i) used[m9[i]] = 1;
        for (unsigned v = 1; v < 512; ++v)
            if (used[v]) {
                index_of[v] = (int)lib.size();
                lib.push_back((uint16_t)v);
            }
        if (lib.empty()) lib.push_back(1);   // a layer with nothing kept
        std::vector<uint8_t> pid(m9.size(), 0), mask(m9.size(), 0);
        for (size_t i = 0; i < m9.size(); ++i)
            if (m9[i]) {
                pid[i] = (uint8_t)index_of[m9[i]];
                mask[i] = 1;
            }
        return pack_impl(w.data(), p->dtype, F, C4, lib.data(), (int)lib.size(), pid.data(), mask.data(),
                         upload ? 0u : (unsigned)PCONV_PACK_HOST_ONLY, true, false, out);
    } catch (const std::bad_alloc&) {
        return PCONV_ENOMEM;
    }
}

extern "C" int pconv_filter_similarity_order(const uint8_t* mask, int F, int C, int group, uint32_t* order_out) {
    if (!mask || !order_out) return PCONV_EINVAL;
    if (int rc = check_fc(F, C)) return rc;
    if (group < 1) return PCONV_EINVAL;
    try {
        // the channels every filter keeps, as bit sets
        const size_t words = ((size_t)C + 63) / 64;
        std::vector<uint64_t> support((size_t)F * words, 0);
        std::vector<uint32_t> count((size_t)F, 0);
        for (int f = 0; f < F; ++f)
            for (int c = 0; c < C; ++c)
                if (mask[(size_t)f * C + c]) {
                    support[(size_t)f * words + (size_t)c / 64] |= 1ull << (c % 64);
                    ++count[(size_t)f];
                }
        std::vector<char> taken((size_t)F, 0);
        std::vector<uint64_t> uni(words);
        int placed = 0;
        while (placed < F) {
            // a group starts with the filter that keeps the most kernels (lowest index among equals) ...
            int seed = -1;
            for (int f = 0; f < F; ++f)
                if (!taken[(size_t)f] && (seed < 0 || count[(size_t)f] > count[(size_t)seed])) seed = f;
            taken[(size_t)seed] = 1;
            order_out[placed++] = (uint32_t)seed;
            std::copy(support.begin() + (size_t)seed * words, support.begin() + (size_t)(seed + 1) * words, uni.begin());
            // ... and takes, one at a time, the filter that adds the fewest channels to the group's union; among
            // equals the one that shares the most with it, then the lowest index
            for (int k = 1; k < group && placed < F; ++k) {
                int best = -1;
                uint32_t best_add = 0, best_share = 0;
                for (int f = 0; f < F; ++f) {
                    if (taken[(size_t)f]) continue;
                    uint32_t add = 0, share = 0;
                    const uint64_t* sf = &support[(size_t)f * words];
                    for (size_t w = 0; w < words; ++w) {
                        add += (uint32_t)__builtin_popcountll(sf[w] & ~uni[w]);
                        share += (uint32_t)__builtin_popcountll(sf[w] & uni[w]);
                    }
                    if (best < 0 || add < best_add || (add == best_add && share > best_share)) {
                        best = f;
                        best_add = add;
                        best_share = share;
                    }
                }
                taken[(size_t)best] = 1;
                order_out[placed++] = (uint32_t)best;
                const uint64_t* sb = &support[(size_t)best * words];
                for (size_t w = 0; w < words; ++w) uni[w] |= sb[w];
            }
        }
    } catch (const std::bad_alloc&) {
        return PCONV_ENOMEM;
    }
    return PCONV_OK;
}

extern "C" int pconv_packed_mfma_blocks(const pconv_packed* p, int tile_filters, int* listed_blocks, int* all_blocks) {
    if (!p) return PCONV_EINVAL;
    for (const pconv::MfmaWeights& m : p->mfma)
        if (m.mt == tile_filters) {
            if (listed_blocks) *listed_blocks = m.total_blocks;
            if (all_blocks) *all_blocks = m.n_mtiles * m.n_cblocks;
            return PCONV_OK;
        }
    return PCONV_EUNSUPPORTED;
}

extern "C" int pconv_packed_parity_form(const pconv_packed* p, int pad, pconv_packed** out) {
    return pconv::derive_for_stride2(p, pad, false, out);
}

extern "C" int pconv_packed_library(const pconv_packed* p, uint16_t* lib_out) {
    if (!p || !lib_out) return PCONV_EINVAL;
    std::memcpy(lib_out, p->lib.data(), p->lib.size() * sizeof(uint16_t));
    return PCONV_OK;
}

extern "C" int pconv_packed_export(const pconv_packed* p, uint32_t* filter_order, uint32_t* grp_ptr, uint16_t* cin,
                                   void* w4, size_t* n_kept) {
    if (!p) return PCONV_EINVAL;
    if (filter_order) std::memcpy(filter_order, p->filter_order.data(), p->filter_order.size() * sizeof(uint32_t));
    if (grp_ptr) std::memcpy(grp_ptr, p->grp_ptr.data(), p->grp_ptr.size() * sizeof(uint32_t));
    if (cin && !p->cin.empty()) std::memcpy(cin, p->cin.data(), p->cin.size() * sizeof(uint16_t));
    if (w4 && !p->w4.empty()) std::memcpy(w4, p->w4.data(), p->w4.size());
    if (n_kept) *n_kept = p->n_kept;
    return PCONV_OK;
}

// The inverse of pconv_packed_export: the canonical arrays are checked, spread back into a dense masked tensor with its
// pattern ids and connectivity mask, and packed again, so that an imported layer is in every respect the layer that
// pconv_pack would have made from the original weights.
extern "C" int pconv_packed_import(const uint32_t* filter_order, const uint32_t* grp_ptr, const uint16_t* cin,
                                   const void* w4, int dtype, int F, int C, const uint16_t* lib, int K,
                                   unsigned flags, pconv_packed** out) {
    if (!out) return PCONV_EINVAL;
    *out = nullptr;
    if (!filter_order || !grp_ptr) return PCONV_EINVAL;
    if (dtype != PCONV_F32 && dtype != PCONV_F16) return PCONV_EINVAL;
    if (int rc = check_library(lib, K)) return rc;
    if (int rc = check_fc(F, C)) return rc;
    const size_t esize = dtype == PCONV_F16 ? 2 : 4;
    const size_t n_groups = (size_t)F * K;
    const size_t n_kept = grp_ptr[n_groups];
    if (grp_ptr[0] != 0 || n_kept > (size_t)F * C) return PCONV_EINVAL;
    for (size_t g = 0; g < n_groups; ++g)
        if (grp_ptr[g] > grp_ptr[g + 1]) return PCONV_EINVAL;
    if (n_kept && (!cin || !w4)) return PCONV_EINVAL;
    try {
        std::vector<unsigned char> seen((size_t)F, 0);
        for (int i = 0; i < F; ++i) {
            if (filter_order[i] >= (uint32_t)F || seen[filter_order[i]]) return PCONV_EINVAL;
            seen[filter_order[i]] = 1;
        }
        std::vector<int> taps((size_t)K * 4);
        for (int j = 0; j < K; ++j) {
            int n = 0;
            for (int t = 0; t < 9; ++t)
                if (lib[j] >> t & 1) taps[(size_t)j * 4 + n++] = t;
        }
        std::vector<unsigned char> w((size_t)F * C * 9 * esize, 0);
        std::vector<uint8_t> pid((size_t)F * C, 0), mask((size_t)F * C, 0);
        const unsigned char* src = static_cast<const unsigned char*>(w4);
        for (int i = 0; i < F; ++i) {
            const size_t f = filter_order[i];
            for (int j = 0; j < K; ++j) {
                const size_t a = grp_ptr[(size_t)i * K + j], b = grp_ptr[(size_t)i * K + j + 1];
                for (size_t e = a; e < b; ++e) {
                    const size_t c = cin[e];
                    // inside a group channels ascend; over the groups of a filter no channel comes twice
                    if (c >= (size_t)C || (e > a && cin[e - 1] >= c) || mask[f * C + c]) return PCONV_EINVAL;
                    mask[f * C + c] = 1;
                    pid[f * C + c] = (uint8_t)j;
                    for (int k = 0; k < 4; ++k)
                        std::memcpy(&w[((f * C + c) * 9 + taps[(size_t)j * 4 + k]) * esize], src + (e * 4 + k) * esize,
                                    esize);
                }
            }
        }
        return pack_impl(w.data(), dtype, F, C, lib, K, pid.data(), mask.data(), flags, false, true, out);
    } catch (const std::bad_alloc&) {
        return PCONV_ENOMEM;
    }
}

// The balanced order of one tiling: as it lies on the device, or as it was or would be found on the host.
static int staging_order(const pconv_packed* p, const pconv::BalancedLayout& b, std::vector<uint32_t>* perm) {
    if (b.d_perm) return pconv::download_order(b, perm);
    pconv::BalancedLayout found = b;
    if (found.perm.empty()) find_balanced(p, &found);
    *perm = found.perm;
    return PCONV_OK;
}

extern "C" int pconv_packed_order(const pconv_packed* p, int waves, int filters_per_wave, int channels, uint32_t* order_out,
                                  size_t* positions) {
    if (!p) return PCONV_EINVAL;
    for (const pconv::BalancedLayout& b : p->balanced) {
        if (b.fw != waves || b.nf != filters_per_wave || b.cc != channels) continue;
        if (positions) *positions = (size_t)b.n_groups * b.n_chunks * b.cc;
        if (!order_out) return PCONV_OK;
        try {
            std::vector<uint32_t> perm;
            if (int rc = staging_order(p, b, &perm)) return rc;
            std::copy(perm.begin(), perm.end(), order_out);
        } catch (const std::bad_alloc&) {
            return PCONV_ENOMEM;
        }
        return PCONV_OK;
    }
    return PCONV_EUNSUPPORTED;
}

extern "C" int pconv_packed_balance(const pconv_packed* p, int waves, int filters_per_wave, int balanced,
                                    double* mean_per_wave, double* mean_of_max) {
    if (!p || !mean_per_wave || !mean_of_max) return PCONV_EINVAL;
    if (waves < 1 || filters_per_wave < 1) return PCONV_EINVAL;
    const int F = p->F, fg = waves * filters_per_wave, cc = 32;
    const pconv::BalancedLayout* bl = nullptr;
    for (const pconv::BalancedLayout& b : p->balanced)
        if (b.fw == waves && b.nf == filters_per_wave && b.cc == cc) bl = &b;
    if (balanced && !bl) return PCONV_EUNSUPPORTED;
    std::vector<uint32_t> pos_of;                            // [group][C]: position of a channel in its group's order
    if (balanced) {
        try {
            std::vector<uint32_t> perm;
            if (int rc = staging_order(p, *bl, &perm)) return rc;
            const int npos = bl->n_chunks * cc;
            pos_of.assign((size_t)bl->n_groups * p->C, 0);
            for (size_t at = 0; at < perm.size(); ++at)
                if (perm[at] != pconv::kNoChannel) {
                    if (perm[at] >= (uint32_t)p->C) return PCONV_ESTATE;
                    pos_of[at / npos * p->C + perm[at]] = (uint32_t)(at % npos);
                }
        } catch (const std::bad_alloc&) {
            return PCONV_ENOMEM;
        }
    }
    const int nch = balanced ? bl->n_chunks : (p->C + cc - 1) / cc;
    // kept kernels of (filter position, chunk of 32 staged channels), from the canonical arrays
    std::vector<uint32_t> counts;
    try {
        counts.assign((size_t)F * nch, 0);
    } catch (const std::bad_alloc&) {
        return PCONV_ENOMEM;
    }
    for (int i = 0; i < F; ++i)
        for (uint32_t e = p->grp_ptr[(size_t)i * p->K]; e < p->grp_ptr[(size_t)(i + 1) * p->K]; ++e) {
            const uint32_t at = balanced ? pos_of[(size_t)(i / fg) * p->C + p->cin[e]] : p->cin[e];
            ++counts[(size_t)i * nch + at / cc];
        }
    auto count = [&](int pos, int k) -> uint32_t { return counts[(size_t)pos * nch + k]; };
    double sum = 0.0, sum_max = 0.0;
    long long n_wave_chunks = 0, n_chunks = 0;
    for (int g = 0; g * fg < F; ++g)
        for (int k = 0; k < nch; ++k) {
            uint32_t mx = 0;
            for (int w = 0; w < waves; ++w) {
                uint32_t load = 0;
                for (int a = 0; a < filters_per_wave; ++a) {
                    const int pos = g * fg + w + a * waves;
                    if (pos < F) load += count(pos, k);
                }
                mx = std::max(mx, load);
                sum += load;
                ++n_wave_chunks;
            }
            sum_max += mx;
            ++n_chunks;
        }
    *mean_per_wave = n_wave_chunks ? sum / (double)n_wave_chunks : 0.0;
    *mean_of_max = n_chunks ? sum_max / (double)n_chunks : 0.0;
    return PCONV_OK;
}

extern "C" int pconv_packed_stats(const pconv_packed* p, int* F, int* C, int* K, int* dtype, size_t* n_kept) {
    if (!p) return PCONV_EINVAL;
    if (F) *F = p->F;
    if (C) *C = p->C;
    if (K) *K = p->K;
    if (dtype) *dtype = p->dtype;
    if (n_kept) *n_kept = p->n_kept;
    return PCONV_OK;
}

extern "C" void pconv_free(pconv_packed* p) {
    if (!p) return;
    for (pconv_packed*& child : p->by_parity) {
        pconv_free(child);
        child = nullptr;
    }
    pconv::release_device(p);
    delete p;
}

extern "C" const char* pconv_strerror(int code) {
    switch (code) {
        case PCONV_OK: return "ok";
        case PCONV_EINVAL: return "invalid argument (null pointer, bad enum or flag)";
        case PCONV_EPATTERN: return "bad pattern library or pattern id (masks need exactly four of nine bits, 1 <= K <= 126, id < K)";
        case PCONV_ESHAPE: return "bad shape (non-positive extent, C >= 65536, empty output or size overflow)";
        case PCONV_EUNSUPPORTED: return "unsupported stride (1 or 2) or pad (0 or 1)";
        case PCONV_ENOMEM: return "out of memory";
        case PCONV_EHIP: return "HIP runtime error (see pconv_last_hip_error)";
        case PCONV_ESTATE: return "packed handle has no device copy (packed host-only), belongs to another device, or lacks a form of the layer that only an allocating call can build";
        case PCONV_ESCRATCH: return "the launch needs more scratch memory than the fixed arena of pconv_conv3x3_noalloc holds";
        default: return "unknown pconv error code";
    }
}
