// Masked tree attention over a segmented KV cache (paper Sections 3.4 and 3.5, Appendix A.1
// and A.2): what stands between the q/k/v projections and the o projection of a decoding step
// that carries several output streams and, per stream, a draft tree with forecast embeddings.
//
// A block takes up to 16 or 32 query vectors of one stream and one kv head.  All keys these rows may see lie on one
// axis (forecast prefix, prefill, the stream's own segment, the rows of the step), cut into chunks of 32, and the
// block's waves take chunks in turn.  A wave works by itself: no barrier, no data of other waves, until the waves'
// results are merged through LDS at the end.  Where the keys are more than one block per query tile gets through in
// good time, several blocks share the axis, and a second kernel merges what they leave in the workspace.
//
// Scores are K . Q^T on the matrix units (16x16x32 bf16, fp32 accumulation): a lane then holds eight keys of ONE query
// vector, its maximum and rescaling are scalars, and its weights, as two bf16 halves (nothing is rounded to 8
// bits), are where O^T += V^T . P^T wants them if the keys of that product are counted in the same order.  Values go
// through a wave-private piece of LDS, which transposes them on the way out (ds_read_b64_tr_b16).  Everything is merged
// in a fixed order: results are reproducible.
//
// What bounds a call of decoding size is the chain of trips to memory and the cold fetch of the code, so there is one
// launch where that does, and the loop's body exists once and is short; a long call is bound by what the caches hand
// out, and by the vector work of the weights.  A block per chunk run and segment with keys and values shared through LDS,
// and always a second kernel, was: 8 streams x 4 rows, 32 query heads on 8 kv heads of 64 features, 2048 keys 13.0 ->
// 9.4 us; 85 keys of one head 6.5 -> 3.5; 17576 keys of 8 heads, 120 query vectors per stream, 87 -> 44; 333 keys
// of 128 features, 13 streams x 168 query vectors, 39.6 -> 16.5.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

#include "../../include/mlora_tree_attention.h"

namespace mlora {

namespace {

constexpr int KC = 32;                   // keys per chunk
constexpr float NEG_BIG = -1.0e30f;      // "no key seen yet"
constexpr float UNSEEN = -3.0e38f;       // score of a key that is not visible: exp2(UNSEEN - NEG_BIG) is 0

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

struct AttnArgs {
    const uint16_t *q;                   // bf16 [M][Hq][D]
    const uint16_t *k_prefill, *v_prefill, *k_fprefix, *v_fprefix, *k_stream, *v_stream, *k_new, *v_new;
    const int *len_stream, *parent;
    const uint8_t *is_forecast;
    float *part_out;                     // several blocks per query tile: [splits][S * R * Hq][D], not normalised
    float2 *part_ml;                     // [splits][S * R * Hq]: maximum (of scores in units of log 2) and sum
    void *out;
    int Hq, Hkv, G, S, R, M;
    int Lp, Lf, cap;
    int splits;                          // blocks that share the keys of a query tile
    unsigned g_inv;                      // ceil(2^16 / G): v / G = (v * g_inv) >> 16 for v < 512
    int out_fp32;
    float scale2;                        // scale * log2(e)
};

// LDS of a wave: the values of a chunk on their way to the matrix units, then its share of the result.
template <int D, int QT>
struct WaveLds {
    static constexpr int VROW = D * 2 + 32;              // bytes of a row of values; +32: eight rows cover all banks once
    static constexpr int OROW = D + 4;                   // floats of a query vector's output; +4: 16-byte stores of 16 rows do not collide
    static constexpr int O_BYTES = QT * 16 * OROW * 4, ML_BYTES = QT * 16 * 8;
    static constexpr int BYTES = KC * VROW > O_BYTES + ML_BYTES ? KC * VROW : O_BYTES + ML_BYTES;
};

// a value combined over the four quarters of a wave (lanes 16 and 32 apart); every lane gets the result
template <class Op>
__device__ __forceinline__ float over_quarters(float v, const Op &op)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

template <int D, int QT, int W, bool SPLIT>
__global__ __launch_bounds__(64 * W, (D == 64 && QT == 1 ? 4 : 2)) void tree_attn(const AttnArgs a)
{
    using L = WaveLds<D, QT>;
    constexpr int DK = D / 32, DB = D / 16, VI = KC * D / 512;
    __shared__ __align__(16) unsigned char smem[W * L::BYTES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, lq = lane >> 4;
    const int hk = blockIdx.x;
    const int s = SPLIT ? (int)blockIdx.z / a.splits : (int)blockIdx.z, z = SPLIT ? (int)blockIdx.z - s * a.splits : 0;
    const int n_qv = a.R * a.G, qv0 = (int)blockIdx.y * (16 * QT);

    // the axis of keys: chunks of the forecast prefix, the prefill, the stream's segment, the rows of the step.  (The
    // forecast prefix comes first: a row that may not see it starts afresh behind it, see below.)
    const int len = a.cap > 0 ? max(0, min(a.len_stream[s], a.cap)) : 0;
    const int end_f = (a.Lf + KC - 1) / KC, end_p = end_f + (a.Lp + KC - 1) / KC, end_s = end_p + (len + KC - 1) / KC, chunks = end_s + (a.R + KC - 1) / KC;
    struct Chunk {
        const unsigned char *k, *v;
        int n;                                           // keys, at most KC
        int pitch;                                       // bytes of a row
    };
    auto chunk_of = [&](int c) {
        const uint16_t *kb = a.k_new, *vb = a.v_new;
        int first = (c - end_s) * KC, n = a.R - first, pitch = a.Hkv * D * 2;
        size_t row = (size_t)(s * a.R + first) * a.Hkv + hk;           // in rows of D
        if (c < end_s) {
            pitch = D * 2;
            if (c < end_f)      { kb = a.k_fprefix; vb = a.v_fprefix; first = c * KC; row = (size_t)hk * a.Lf + first; n = a.Lf - first; }
            else if (c < end_p) { kb = a.k_prefill; vb = a.v_prefill; first = (c - end_f) * KC; row = (size_t)hk * a.Lp + first; n = a.Lp - first; }
            else                { kb = a.k_stream; vb = a.v_stream; first = (c - end_p) * KC; row = ((size_t)s * a.Hkv + hk) * a.cap + first; n = len - first; }
        }
        return Chunk{reinterpret_cast<const unsigned char *>(kb + row * D), reinterpret_cast<const unsigned char *>(vb + row * D), min(n, KC), pitch};
    };
    u32x4 kf[KC / 16][DK], vr[VI];
    // keys as A operands: lane (l16, lq) holds features 8 * lq .. of key 16 * t + l16 (past the end: the last key)
    auto load_k = [&](const Chunk &c) {
#pragma unroll
        for (int t = 0; t < KC / 16; ++t) {
            const unsigned at = (unsigned)min(16 * t + l16, c.n - 1) * (unsigned)c.pitch + lq * 16;
#pragma unroll
            for (int kk = 0; kk < DK; ++kk) kf[t][kk] = *reinterpret_cast<const u32x4 *>(c.k + at + kk * 64);
        }
    };
    // values row by row
    auto load_v = [&](const Chunk &c) {
#pragma unroll
        for (int i = 0; i < VI; ++i) {
            const int piece = i * 64 + lane;
            vr[i] = *reinterpret_cast<const u32x4 *>(c.v + (unsigned)min(piece / (D / 8), c.n - 1) * (unsigned)c.pitch + (piece % (D / 8)) * 16);
        }
    };
    int c = z * W + wave;
    const int stride = SPLIT ? a.splits * W : W;
    Chunk cur = chunk_of(min(c, chunks - 1));
    if (c < chunks) {
        load_k(cur);
        load_v(cur);
    }

    // this lane's query vectors (B operands: lane (l16, lq) holds features 8 * lq .. of vector l16 of a tile)
    u32x4 qf[QT][DK];
    int row[QT];
    float m[QT], l[QT];
    f32x4 o[QT][DB];
    bool fc[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        const int v = min(qv0 + 16 * t + l16, n_qv - 1);
        row[t] = (int)((unsigned)v * a.g_inv >> 16);
        const uint16_t *qp = a.q + ((size_t)(s * a.R + row[t]) * a.Hq + hk * a.G + (v - row[t] * a.G)) * D + 8 * lq;
#pragma unroll
        for (int kk = 0; kk < DK; ++kk) qf[t][kk] = *reinterpret_cast<const u32x4 *>(qp + 32 * kk);
        fc[t] = a.Lf > 0 && a.is_forecast[s * a.R + row[t]] != 0;
        m[t] = NEG_BIG;
        l[t] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[t][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    unsigned char *const mine = smem + wave * L::BYTES;
    unsigned char *const v_in = mine + (lane / (D / 8)) * L::VROW + (lane % (D / 8)) * 16;
    using Lds4 = __attribute__((address_space(3))) s16x4;
    const unsigned char *const v_out = mine + (4 * lq + (l16 >> 2)) * L::VROW + (l16 & 3) * 8;

#pragma nounroll
    while (c < chunks) {
        // scores: element e of sc[t][j] is key 16 * j + 4 * lq + e against query vector l16 of tile t
        f32x4 sc[QT][KC / 16];
#pragma unroll
        for (int j = 0; j < KC / 16; ++j)
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                sc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < DK; ++kk) sc[t][j] = mfma16(__builtin_bit_cast(uint4, kf[j][kk]), __builtin_bit_cast(uint4, qf[t][kk]), sc[t][j]);
            }
        // values -> LDS, then the next chunk is on its way while this one is worked on.  (The wave's own LDS accesses are
        // ordered: no barrier.)
#pragma unroll
        for (int k = 0; k < VI; ++k) *reinterpret_cast<u32x4 *>(v_in + k * (512 / D) * L::VROW) = vr[k];
        const int here = c, n = cur.n;
        c += stride;
        if (c < chunks) {
            cur = chunk_of(c);
            load_k(cur);
            load_v(cur);
        }
#pragma unroll
        for (int t = 0; t < QT; ++t)
#pragma unroll
            for (int j = 0; j < KC / 16; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) sc[t][j][e] *= a.scale2;
        // keys some rows may not see: those past the end, the forecast prefix, other branches of the tree
        if (n < KC || here < end_f || here >= end_s) {
            const unsigned keys = ~0u >> (KC - n);
            unsigned anc_lo = 0, anc_hi = 0;
            if (here >= end_s) {
                // lane r: the rows that row r may see, itself and what it continues (a parent must be an earlier row: the
                // walk strictly descends, so it ends and stays in bounds whatever the array holds)
                const int up0 = a.parent[s * a.R + min(lane, a.R - 1)];
                int r = lane < a.R ? lane : -1;
                while (__ballot(r >= 0)) {
                    if (r >= 0) {
                        anc_lo |= r < 32 ? 1u << r : 0u;
                        anc_hi |= r >= 32 ? 1u << (r - 32) : 0u;
                    }
                    const int up = __shfl(up0, max(r, 0));
                    r = r >= 0 && up < r ? up : -1;
                }
            }
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                unsigned see = keys;
                if (here >= end_s) see &= (unsigned)__shfl((int)(here == end_s ? anc_lo : anc_hi), row[t]);
                if (here < end_f && !fc[t]) see = 0;
                see >>= 4 * lq;
#pragma unroll
                for (int j = 0; j < KC / 16; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sc[t][j][e] = (see >> (16 * j + e)) & 1 ? sc[t][j][e] : UNSEEN;
            }
        }
        // running maximum and sum (the sum of the lane's own keys), weights as two bf16 halves
        uint4 ph[QT], pl[QT];
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            float top = m[t];
#pragma unroll
            for (int j = 0; j < KC / 16; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) top = fmaxf(top, sc[t][j][e]);
            top = over_quarters(top, [](float x, float y) { return fmaxf(x, y); });
            const float keep = __builtin_amdgcn_exp2f(m[t] - top);      // (1 while nothing has been seen)
            m[t] = top;
            float sum = 0.f;
            uint32_t h[4], w[4];
#pragma unroll
            for (int j = 0; j < KC / 16; ++j) {
                float p[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    p[e] = __builtin_amdgcn_exp2f(sc[t][j][e] - top);
                    sum += p[e];
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    h[2 * j + i] = pack_bf16(p[2 * i], p[2 * i + 1]);
                    w[2 * j + i] = pack_bf16(p[2 * i] - bf16_bits_to_float(h[2 * j + i] & 0xFFFFu), p[2 * i + 1] - __uint_as_float(h[2 * j + i] & 0xFFFF0000u));
                }
            }
            l[t] = l[t] * keep + sum;
#pragma unroll
            for (int db = 0; db < DB; ++db) o[t][db] *= keep;
            ph[t] = make_uint4(h[0], h[1], h[2], h[3]);
            pl[t] = make_uint4(w[0], w[1], w[2], w[3]);
        }
        // place 8 * lq + 4 * h + e of the product is key 16 * h + 4 * lq + e, as in the scores.
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lds4 *)(v_out + db * 32)));
            const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((Lds4 *)(v_out + 16 * L::VROW + db * 32)));
            const uint4 vf = make_uint4(lo.x, lo.y, hi.x, hi.y);
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                o[t][db] = mfma16(vf, ph[t], o[t][db]);
                o[t][db] = mfma16(vf, pl[t], o[t][db]);
            }
        }
        // a row that may not see the forecast prefix has seen nothing yet (whatever the values there are)
        if (here < end_f) {
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                m[t] = fc[t] ? m[t] : NEG_BIG;
                l[t] = fc[t] ? l[t] : 0.f;
#pragma unroll
                for (int db = 0; db < DB; ++db) o[t][db] = fc[t] ? o[t][db] : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
    }

    // the waves' results, merged in the order of the waves
    const int waves = min(W, chunks - z * W);                  // with at least one chunk (a split's last blocks may have none)
    if (wave < waves) {
        float *const om = reinterpret_cast<float *>(mine);
        float2 *const ml = reinterpret_cast<float2 *>(mine + L::O_BYTES);
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            const float sum = over_quarters(l[t], [](float x, float y) { return x + y; });
            if (lq == 0) ml[16 * t + l16] = make_float2(m[t], sum);
#pragma unroll
            for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4 *>(om + (16 * t + l16) * L::OROW + 16 * db + 4 * lq) = o[t][db];
        }
    }
    __syncthreads();
    for (int i = tid; i < QT * 16 * (D / 4); i += 64 * W) {
        const int qv = i / (D / 4), f = i % (D / 4) * 4, v = qv0 + qv;
        if (v >= n_qv) break;
        auto ml_of = [&](int w) { return reinterpret_cast<const float2 *>(smem + w * L::BYTES + L::O_BYTES)[qv]; };
        float top = NEG_BIG;
#pragma unroll 4
        for (int w = 0; w < waves; ++w) top = fmaxf(top, ml_of(w).x);
        f32x4 num = {0.f, 0.f, 0.f, 0.f};
        float den = 0.f;
#pragma unroll 4
        for (int w = 0; w < waves; ++w) {
            const float2 x = ml_of(w);
            const float weight = __builtin_amdgcn_exp2f(x.x - top);
            num += weight * *reinterpret_cast<const f32x4 *>(smem + w * L::BYTES + (qv * L::OROW + f) * 4);
            den += weight * x.y;
        }
        const int r = (int)((unsigned)v * a.g_inv >> 16);
        const size_t vec = (size_t)(s * a.R + r) * a.Hq + hk * a.G + (v - r * a.G);
        if constexpr (SPLIT) {
            const size_t at = (size_t)z * a.M * a.Hq + vec;
            if (f == 0) a.part_ml[at] = make_float2(top, den);
            *reinterpret_cast<f32x4 *>(a.part_out + at * D + f) = num;
        } else {
            num /= den;                                        // (a row always sees itself: den > 0)
            if (a.out_fp32) *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(a.out) + vec * D + f) = num;
            else *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(a.out) + vec * D + f) = make_uint2(pack_bf16(num[0], num[1]), pack_bf16(num[2], num[3]));
        }
    }
}

// Four features of a query vector per thread: merge what the blocks that shared its keys saw, in their order.
template <int D>
__global__ __launch_bounds__(256) void tree_attn_combine(const AttnArgs a)
{
    const int i = (int)blockIdx.x * 256 + (int)threadIdx.x, vecs = a.M * a.Hq;
    if (i >= vecs * (D / 4)) return;
    const int vec = i / (D / 4), f = i % (D / 4) * 4;
    constexpr int RB = 8;                                      // results per trip to memory
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f, run_top = NEG_BIG;
    for (int z0 = 0; z0 < a.splits; z0 += RB) {
        float2 ml[RB];
        f32x4 pv[RB];
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const size_t at = (size_t)min(z0 + u, a.splits - 1) * vecs + vec;
            ml[u] = a.part_ml[at];
            pv[u] = *reinterpret_cast<const f32x4 *>(a.part_out + at * D + f);
        }
        float top = run_top;
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            if (z0 + u >= a.splits) ml[u] = make_float2(NEG_BIG, 0.f), pv[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            top = fmaxf(top, ml[u].x);
        }
        const float keep = __builtin_amdgcn_exp2f(run_top - top);
        num *= keep;
        den *= keep;
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const float w = __builtin_amdgcn_exp2f(ml[u].x - top);
            num += w * pv[u];
            den += w * ml[u].y;
        }
        run_top = top;
    }
    num /= den;
    const size_t at = (size_t)vec * D + f;
    if (a.out_fp32) *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(a.out) + at) = num;
    else *reinterpret_cast<uint2 *>(reinterpret_cast<uint16_t *>(a.out) + at) = make_uint2(pack_bf16(num[0], num[1]), pack_bf16(num[2], num[3]));
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// What a workspace is sized for: a partial result per query vector for every run of chunks of 64 keys (about 128 blocks for the
// longest segment, at most 16 chunks in a run) of each segment, and one for the rows of the step.
constexpr int RUN_KC = 64;
int runs_of(int len, int chunks_per_run) { return ((len + RUN_KC - 1) / RUN_KC + chunks_per_run - 1) / chunks_per_run; }
int most_splits(const mlora_tree_attn &t)
{
    const int longest = std::max(std::max(t.len_prefill, t.cap_stream), t.len_fprefix);
    const long long cpr = ((long long)(longest + RUN_KC - 1) / RUN_KC * t.n_kv_heads + 127) / 128;
    const int n = cpr < 1 ? 1 : cpr > 16 ? 16 : (int)cpr;
    return runs_of(t.len_prefill, n) + runs_of(t.len_fprefix, n) + runs_of(t.cap_stream, n) + 1;
}
size_t workspace_floats(const mlora_tree_attn &t)
{
    return (size_t)most_splits(t) * t.n_q_heads * (size_t)t.n_streams * t.rows_per_stream * ((size_t)t.head_dim + 2);
}

// How a call is cut.  Lines drawn from 140 calls (1 to 14 streams, 1 to 312 query vectors of a stream and kv head, 1
// to 24000 keys), each with one and two tiles, 4 and 8 waves, 1 to 32 splits; the figures are us in a graph.
struct Plan {
    int tiles;                           // query tiles (of 16) of a block
    int waves;                           // of a block
    int splits;                          // blocks that share the keys of a query tile
};
Plan plan_of(const mlora_tree_attn &t)
{
    Plan p;
    const bool wide = t.head_dim == 128;
    const int qv = t.rows_per_stream * (t.n_q_heads / t.n_kv_heads);
    const int chunks = (t.len_fprefix + KC - 1) / KC + (t.len_prefill + KC - 1) / KC + (t.cap_stream + KC - 1) / KC + (t.rows_per_stream + KC - 1) / KC;
    const long long heads = (long long)t.n_kv_heads * t.n_streams, tiles16 = (qv + 15) / 16;
    // Two tiles per block halve what the caches hand out, but a wave's work is twice as long and fewer of them are
    // resident: they pay where one tile per block would read more than 50 MB of keys and values (288 blocks of 33
    // chunks: 12.7 -> 9.7; 96 of 33 chunks: 8.1 -> 9.5).
    p.tiles = qv > 16 && heads * tiles16 * chunks * (KC * 4ll * t.head_dim) > 50000000 ? 2 : 1;
    const long long blocks = heads * ((tiles16 + p.tiles - 1) / p.tiles);
    // Shared keys cost a second launch (2 to 3 us) and pay from about 30 chunks on (20 of 128 features): 8 blocks of 33
    // chunks 7.6 -> 5.7, of 23 chunks 6.5 -> 6.7.  Up to a block per compute unit, and up to 8 of them if no wave has
    // more than ten chunks; in long calls (150 chunks) two smaller blocks per compute unit (144 blocks of 510 chunks:
    // 75 -> 56), but one where two tiles of 128 features fill the registers.
    long long splits = 1;
    if (chunks >= 150) {
        splits = std::min(16ll, (wide && p.tiles == 2 && blocks <= 100 ? 256 : 512) / blocks);
    } else if (chunks >= (wide ? 20 : 28)) {
        splits = std::min(256 / blocks, (long long)std::min(chunks / 4, std::max(8, chunks / 10)));
    }
    splits = std::min(splits, (long long)most_splits(t));
    if (splits > 8 && splits < 12) splits = 8;             // (what the merging kernel asks for at once)
    p.splits = (int)std::max(1ll, splits);
    // Eight waves where four would have more than four chunks each (three; one of 128 features) and the blocks find room.
    if (p.splits > 1) p.waves = chunks < 150 && chunks > 16 * p.splits ? 8 : 4;
    else              p.waves = chunks > (wide ? 4 : 12) && blocks <= (wide ? 256 : 512) ? 8 : 4;
    return p;
}

mlora_status check(const mlora_tree_attn *t)
{
    if (!t) return MLORA_EINVAL;
    if (t->head_dim != 64 && t->head_dim != 128) return MLORA_ESHAPE;
    if (t->n_kv_heads <= 0 || t->n_q_heads <= 0 || t->n_q_heads % t->n_kv_heads != 0) return MLORA_ESHAPE;
    if (t->n_q_heads / t->n_kv_heads > 8 || t->n_q_heads > 65535 || t->n_kv_heads > 65535) return MLORA_ESHAPE;
    if (t->n_streams <= 0 || t->rows_per_stream <= 0 || t->rows_per_stream > 64) return MLORA_ESHAPE;
    if ((long long)t->n_streams * t->rows_per_stream > MLORA_MAX_ROWS) return MLORA_ESHAPE;
    if (t->len_prefill < 0 || t->len_fprefix < 0 || t->cap_stream < 0) return MLORA_ESHAPE;
    if (t->len_prefill > (1 << 24) || t->len_fprefix > (1 << 24) || t->cap_stream > (1 << 24)) return MLORA_ESHAPE;
    if (!t->k_new || !t->v_new || !t->parent || !t->is_forecast) return MLORA_EINVAL;
    if (t->len_prefill > 0 && (!t->k_prefill || !t->v_prefill)) return MLORA_EINVAL;
    if (t->len_fprefix > 0 && (!t->k_fprefix || !t->v_fprefix)) return MLORA_EINVAL;
    if (t->cap_stream > 0 && (!t->k_stream || !t->v_stream || !t->len_stream)) return MLORA_EINVAL;
    const void *ptrs[] = {t->k_prefill, t->v_prefill, t->k_fprefix, t->v_fprefix, t->k_stream, t->v_stream, t->k_new, t->v_new};
    for (const void *p : ptrs)
        if (p && !aligned16(p)) return MLORA_EALIGN;
    if ((reinterpret_cast<uintptr_t>(t->parent) & 3u) || (t->len_stream && (reinterpret_cast<uintptr_t>(t->len_stream) & 3u)))
        return MLORA_EALIGN;
    return MLORA_OK;
}

}  // namespace
}  // namespace mlora

using namespace mlora;

extern "C" {

size_t mlora_tree_attention_workspace_bytes(const mlora_tree_attn *t)
{
    if (check(t) != MLORA_OK) return 0;
    return workspace_floats(*t) * sizeof(float) + 256;
}

mlora_status mlora_tree_attention_plan(const mlora_tree_attn *t, int32_t *info)
{
    if (!info) return MLORA_EINVAL;
    const mlora_status st = check(t);
    if (st != MLORA_OK) return st;
    const Plan p = plan_of(*t);
    info[0] = p.tiles;
    info[1] = p.waves;
    info[2] = p.splits;
    return MLORA_OK;
}

mlora_status mlora_tree_attention(const mlora_tree_attn *t, const void *q, void *out, int32_t out_dtype,
                                  void *workspace, size_t workspace_bytes, void *stream)
{
    const mlora_status st = check(t);
    if (st != MLORA_OK) return st;
    if (!q || !out) return MLORA_EINVAL;
    if (out_dtype != MLORA_Y_BF16 && out_dtype != MLORA_Y_FP32) return MLORA_EINVAL;
    if (!aligned16(q) || !aligned16(out)) return MLORA_EALIGN;
    const size_t need = workspace_floats(*t) * sizeof(float) + 256;
    if (!workspace || workspace_bytes < need) return MLORA_EWORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return MLORA_EALIGN;
    const Plan p = plan_of(*t);

    AttnArgs a;
    a.q = reinterpret_cast<const uint16_t *>(q);
    a.k_prefill = reinterpret_cast<const uint16_t *>(t->k_prefill);
    a.v_prefill = reinterpret_cast<const uint16_t *>(t->v_prefill);
    a.k_fprefix = reinterpret_cast<const uint16_t *>(t->k_fprefix);
    a.v_fprefix = reinterpret_cast<const uint16_t *>(t->v_fprefix);
    a.k_stream = reinterpret_cast<const uint16_t *>(t->k_stream);
    a.v_stream = reinterpret_cast<const uint16_t *>(t->v_stream);
    a.k_new = reinterpret_cast<const uint16_t *>(t->k_new);
    a.v_new = reinterpret_cast<const uint16_t *>(t->v_new);
    a.len_stream = t->len_stream;
    a.parent = t->parent;
    a.is_forecast = t->is_forecast;
    a.out = out;
    a.Hq = t->n_q_heads;
    a.Hkv = t->n_kv_heads;
    a.G = t->n_q_heads / t->n_kv_heads;
    a.S = t->n_streams;
    a.R = t->rows_per_stream;
    a.M = a.S * a.R;
    a.Lp = t->len_prefill;
    a.Lf = t->len_fprefix;
    a.cap = t->cap_stream;
    a.splits = p.splits;
    a.part_out = reinterpret_cast<float *>(workspace);
    a.part_ml = reinterpret_cast<float2 *>(a.part_out + (size_t)p.splits * a.M * a.Hq * t->head_dim);
    a.g_inv = (65536u + (unsigned)a.G - 1) / (unsigned)a.G;
    a.out_fp32 = out_dtype == MLORA_Y_FP32;
    a.scale2 = t->scale * 1.44269504088896340736f;

    hipStream_t s = (hipStream_t)stream;
    const dim3 grid((unsigned)a.Hkv, (unsigned)((a.R * a.G + 16 * p.tiles - 1) / (16 * p.tiles)), (unsigned)(a.S * p.splits));
    auto go = [&](auto d, auto tiles, auto waves) {
        constexpr int D = decltype(d)::value, QT = decltype(tiles)::value, W = decltype(waves)::value;
        if (p.splits == 1) {
            tree_attn<D, QT, W, false><<<grid, dim3(64 * W), 0, s>>>(a);
        } else {
            tree_attn<D, QT, W, true><<<grid, dim3(64 * W), 0, s>>>(a);
            tree_attn_combine<D><<<dim3((unsigned)((a.M * a.Hq * (D / 4) + 255) / 256)), dim3(256), 0, s>>>(a);
        }
    };
    auto by_waves = [&](auto d, auto tiles) {
        if (p.waves == 8) go(d, tiles, std::integral_constant<int, 8>{});
        else              go(d, tiles, std::integral_constant<int, 4>{});
    };
    auto by_tiles = [&](auto d) {
        if (p.tiles == 1) by_waves(d, std::integral_constant<int, 1>{});
        else              by_waves(d, std::integral_constant<int, 2>{});
    };
    if (t->head_dim == 64) by_tiles(std::integral_constant<int, 64>{});
    else                   by_tiles(std::integral_constant<int, 128>{});
    return hipGetLastError() == hipSuccess ? MLORA_OK : MLORA_EHIP;
}

}  // extern "C"
