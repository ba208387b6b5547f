// verify_attention.hip -- multi-query paged GQA attention of the speculative
// verify pass (paper Sec. 2.2: the target model scores every proposed token
// of every request in one pass; Sec. 3.1: the per-step verification cost is
// what decides whether speculation pays off at large batch).
//
// Work decomposition.  A work item is (request i, KV head g, row group, split
// s): the rows are the G * n_i query rows (G = Hq/Hkv q-heads sharing KV head
// g, times the n_i = k_i + 1 positions of the request), the split is a run of
// consecutive 16-token KV blocks.  One workgroup of four wavefronts handles a
// work item; its wavefronts take the split's blocks round-robin, each keeps an
// online-softmax state (running max, running sum, unnormalised output) per row,
// and the four states are merged through LDS at the end.  A request whose keys
// fit one split writes its output directly; otherwise every split writes its
// partial output, maximum and sum, and attn_combine merges them.  (This is the
// fp32 kernel's; the bf16 walk below cuts the work in its own way.)
//
// Masks.  Row j of request i sits at position p = S_i - n_i + j and sees keys
// t <= p, and with a sliding window W only t > p - W; the walk covers the
// union of the rows' visible blocks only.
#include <atomic>
#include <cmath>
#include <type_traits>

#include "common.h"

// m0 is set inside the global->LDS load sequence (see dma16_run); the compiler
// reloads m0 before each of its own uses, so clobbering it there is safe.
#pragma clang diagnostic ignored "-Winline-asm"

namespace averify {
namespace {

constexpr int kAttnWaves = 4;
constexpr int kAttnThreads = kAttnWaves * kWave;
constexpr float kLog2e = 1.4426950408889634f;

struct AttnArgs {
    const void* q;
    const void* kc;
    const void* vc;
    const int32_t* block_tables;
    const int32_t* seq_lens;
    const int32_t* q_start;
    void* out;
    float* part_o;    // [total_q][Hq][max_splits][D] partial outputs, sums of 2^(score - m) v
    float* part_ml;   // [total_q][Hq][max_splits][2] each split's maximum m and sum of 2^(score - m)
    const float* sinks;  // [Hq] sink logits (natural-log units) or null
    const void* k_new;   // fused append: [total_q][Hkv][D] new keys and values, or null
    const void* v_new;
    int num_seqs, hq, hkv, group, max_blocks, num_blocks, window, max_seq_len;
    float scale_log2;  // softmax scale * log2(e): scores live in the log2 domain
    int split_blocks, max_splits, row_groups, rows_per_group;
    int split0;  // first split of the launch
};

// A head's attention sink is one more logit in each row's softmax with a zero
// value: it adds 2^(sink log2(e) - m) to the row's denominator, with m the
// maximum the row's sums are relative to (0 without sinks; for a row with no
// key, m = -inf makes it infinite and the output 0).
__device__ __forceinline__ float sink_term(const float* sinks, int h, float m) {
    return sinks ? exp2f(sinks[h] * kLog2e - m) : 0.f;
}

// Per-request geometry, recomputed identically by every kernel.
struct SeqGeom {
    int q0, n, S, b_lo, b_hi, nsplit;
    int s_raw;  // seq_lens[i] before clamping: the new tokens sit at s_raw - n .. s_raw - 1
};

__device__ __forceinline__ SeqGeom seq_geom(const AttnArgs& a, int i) {
    SeqGeom g;
    g.q0 = a.q_start[i];
    g.n = a.q_start[i + 1] - g.q0;
    int S = a.seq_lens[i];
    g.s_raw = S;
    S = max(0, min(S, min(a.max_seq_len, a.max_blocks * kBlockTokens)));
    g.S = S;
    const int key_lo = a.window > 0 ? max(0, S - g.n - a.window + 1) : 0;
    g.b_lo = key_lo / kBlockTokens;
    g.b_hi = (S + kBlockTokens - 1) / kBlockTokens;
    const int nb = max(0, g.b_hi - g.b_lo);
    g.nsplit = min(a.max_splits, (nb + a.split_blocks - 1) / a.split_blocks);
    return g;
}

// ------------------------------------------------------------------ fp32 storage
//
// A work item is (request, KV head, row group, split), its four wavefronts take
// the split's blocks round-robin, each with an online softmax of its own, and
// merge through LDS at the end.  Both contractions run on v_mfma_f32_16x16x4_f32
// (fp32 products and sums), in 16-row tiles, RT of them per work item:
//   S^T = K Q^T    A = K (16 keys x 4 dims: one float of key l16 per lane), B =
//                  Q^T; lane 16 lg + l16 takes the 16-byte chunks lg, lg + 4, ...
//                  of its key, so each K load of a wavefront is one contiguous
//                  KiB, straight into operand registers; the result lane holds
//                  keys 4 lg .. 4 lg + 3 of row l16;
//   O^T += V^T P^T A = V^T (dim l16 of a 16-dim tile; a lane's 16 bytes of V^T are
//                  its keys 4 lg .. 4 lg + 3), B = P^T, which the S registers
//                  already are: product j takes key 4 lg + j of every lane group.
// Nothing but the query rows goes through LDS.  The next block's K loads leave
// once the scores are done and its V loads once the output is, so a wavefront
// always has 8 KiB in flight (D = 128).
// What bounds it: a block costs a SIMD 2048 cycles of products per tile at D =
// 128 against 16 KiB of K and V, so HBM up to about two tiles, the fp32 products
// beyond.  Against the vector kernel before it (eight rows per work item, each
// walking the keys again): 16 requests of 1k to 8k tokens, 20 rows, 604 MB 604 ->
// 155 us (3.9 TB/s); 8 requests of 2k to 16k tokens, 72 rows 1411 -> 316 us.
// The scores are summed in four chains that are added at the end: shorter sums,
// and no product waits for the one before it.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
// callers' fp32 tensors and the workspace need only be aligned to a float
typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x2u_t __attribute__((ext_vector_type(2), aligned(4)));

// Maximum of v over lanes l, l ^ 16, l ^ 32, l ^ 48 (the four lanes that hold
// one row of an MFMA result tile).  Each permlane swap exchanges half of the
// wavefront between its two operands; with both operands equal to v, the two
// results of lane l are v of l and of l ^ 32 (l ^ 16), in some order.
__device__ __forceinline__ float row_max_4lanes(float v) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const float m = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Softmax weights may exceed 1 by up to this factor (log2) before the stored
// row maximum is raised.
constexpr float kSlackLog2 = 8.f;

// Whether block b has a key that some row of a request must not see: keys past
// its first row's position p_first, or (window) keys below its last row's window.
__device__ __forceinline__ bool block_needs_mask(int b, int p_first, int S, int window) {
    return (b * kBlockTokens + kBlockTokens - 1 > p_first) ||
           (window > 0 && b * kBlockTokens < S - window);
}

// Waves per SIMD that the registers of RT tiles leave room for (an output tile
// takes D / 4 registers, the K and V operands D / 2).
constexpr int f32_waves(int d, int rt) { return d == 64 ? (rt == 1 ? 4 : rt == 2 ? 3 : 2) : rt == 1 ? 3 : 2; }
// Row tiles a work item takes at most: the most that fit 256 registers.
constexpr int f32_max_tiles(int d) { return d == 64 ? 4 : 3; }

// APPEND: the fused KV append (verify_attention_append).  Keys and values of
// the request's new tokens are read from k_new / v_new instead of the cache,
// and the work items of row group 0 (splits cover disjoint blocks) store them
// into the cache as well.
template <int D, int RT, bool APPEND>
__global__ __launch_bounds__(kAttnThreads, f32_waves(D, RT)) void attn_f32(AttnArgs a) {
    constexpr int NU = D / 16;  // 16-byte K chunks per lane; 16-dim output tiles
    constexpr int ROWS = RT * 16;
    constexpr int QN = RT * NU * kWave, MN = kAttnWaves * NU * kWave;

    // Grid (pair within the request + pairs * split, request): workgroups go round
    // the XCDs and their shader engines in launch order, so the heads of a block
    // are read at the same time and the empty splits of short requests come
    // together.  With the split index fastest and a multiple of eight splits an
    // XCD got the same splits of every pair, and the XCDs of the high ones
    // nothing from short requests (16 requests of 1k to 8k tokens, 16 splits:
    // 182 -> 155 us).
    const int i = blockIdx.y;
    const int pairs = a.hkv * a.row_groups;
    const int pair = blockIdx.x % pairs;
    const int s = a.split0 + blockIdx.x / pairs;
    const int kvh = pair / a.row_groups;
    const int rg = pair - kvh * a.row_groups;
    const SeqGeom sg = seq_geom(a, i);
    const int rows_total = a.group * sg.n;
    const int r0 = rg * ROWS;
    if (r0 >= rows_total || s >= sg.nsplit) return;
    const int sb = sg.b_lo + s * a.split_blocks;
    const int se = min(sg.b_hi, sb + a.split_blocks);
    const int tiles = min(RT, (rows_total - r0 + 15) / 16);  // that hold rows

    // the query rows as B operands, one KiB per (tile, chunk); after the walk
    // the wavefronts' outputs of one tile
    __shared__ f32x4_t lds[QN > MN ? QN : MN];
    __shared__ float merge_m[kAttnWaves][ROWS];
    __shared__ float merge_l[kAttnWaves][ROWS];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int l16 = lane & 15, lg = lane >> 4;

    const float* qp = static_cast<const float*>(a.q);
    for (int e = tid; e < QN; e += kAttnThreads) {
        const int rr = r0 + e / (NU * kWave) * 16 + l16;
        const int chunk = lg + 4 * (e / kWave % NU);
        f32x4_t v = {0.f, 0.f, 0.f, 0.f};
        if (rr < rows_total) {
            const int j = rr / a.group, gh = rr - j * a.group;
            v = *reinterpret_cast<const f32x4u_t*>(
                qp + ((int64_t)(sg.q0 + j) * a.hq + kvh * a.group + gh) * D + chunk * 4);
            v *= a.scale_log2;
        }
        lds[e] = v;
    }
    __syncthreads();

    float m[RT], l[RT];
    f32x4_t o[RT][NU];
    int pos[RT], lo[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        m[r] = -INFINITY;
        l[r] = 0.f;
#pragma unroll
        for (int t = 0; t < NU; ++t) o[r][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        pos[r] = sg.S - sg.n + (r0 + r * 16 + l16) / a.group;
        lo[r] = a.window > 0 ? pos[r] - a.window + 1 : 0;
    }

    const float* kc = static_cast<const float*>(a.kc);
    const float* vc = static_cast<const float*>(a.vc);
    const int64_t tile = (int64_t)kBlockTokens * D;
    const int32_t* btab = a.block_tables + (int64_t)i * a.max_blocks;
    // APPEND: new-token positions the walk reaches, and the first row's position
    const int p0 = sg.s_raw - sg.n;
    const int nlo = max(p0, 0), nhi = min(sg.s_raw, sg.S);
    const float* knew = static_cast<const float*>(a.k_new);
    const float* vnew = static_cast<const float*>(a.v_new);
    auto holds_new = [&](int b) { return APPEND && b * kBlockTokens < nhi && (b + 1) * kBlockTokens > nlo; };

    f32x4_t kf[NU], vf[NU];
    auto load_k = [&](int b, int phys) {
        const float* kt = kc + ((int64_t)phys * a.hkv + kvh) * tile + lane * 4;
#pragma unroll
        for (int u = 0; u < NU; ++u) kf[u] = *reinterpret_cast<const f32x4_t*>(kt + u * (kWave * 4));
        if (holds_new(b)) {
            const int tk = b * kBlockTokens + l16;
            if (tk >= nlo && tk < nhi) {
                const float* kn = knew + ((int64_t)(sg.q0 + (tk - p0)) * a.hkv + kvh) * D + lg * 4;
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    kf[u] = *reinterpret_cast<const f32x4u_t*>(kn + u * 16);
                    if (rg == 0) *reinterpret_cast<f32x4_t*>(const_cast<float*>(kt) + u * (kWave * 4)) = kf[u];
                }
            }
        }
    };
    auto load_v = [&](int b, int phys) {
        const float* vt = vc + ((int64_t)phys * a.hkv + kvh) * tile + l16 * kBlockTokens + lg * 4;
#pragma unroll
        for (int t = 0; t < NU; ++t) vf[t] = *reinterpret_cast<const f32x4_t*>(vt + t * (kWave * 4));
        if (holds_new(b)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int tk = b * kBlockTokens + lg * 4 + j;
                if (tk < nlo || tk >= nhi) continue;
                const float* vn = vnew + ((int64_t)(sg.q0 + (tk - p0)) * a.hkv + kvh) * D + l16;
#pragma unroll
                for (int t = 0; t < NU; ++t) {
                    vf[t][j] = vn[t * 16];
                    if (rg == 0) const_cast<float*>(vt)[t * (kWave * 4) + j] = vf[t][j];
                }
            }
        }
    };

    // the ids of the wavefront's next 64 blocks, one per lane; blocks whose id
    // is out of range are left out
    for (int base = sb + w; base < se; base += kAttnWaves * kWave) {
        const int bl = base + kAttnWaves * lane;
        const int id = bl < se ? btab[bl] : -1;
        uint64_t todo = __ballot(id >= 0 && id < a.num_blocks);
        if (todo == 0) continue;
        int at = __builtin_ctzll(todo);
        int phys = __builtin_amdgcn_readlane(id, at);
        int b = base + kAttnWaves * at;
        load_k(b, phys);
        load_v(b, phys);
        while (true) {
            todo &= todo - 1;
            const int at2 = todo ? __builtin_ctzll(todo) : at;
            const int b2 = base + kAttnWaves * at2;
            phys = __builtin_amdgcn_readlane(id, at2);
            const bool masked = block_needs_mask(b, sg.S - sg.n, sg.S, a.window);
            f32x4_t p[RT];
            // keeps the query operands in LDS: hoisted out of the loop they would
            // take D / 4 registers per tile and spill
            int ql = lane;
            asm volatile("" : "+v"(ql));
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                if (r >= tiles) break;
                f32x4_t acc[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const f32x4_t qf = lds[(r * NU + u) * kWave + ql];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[u][e], qf[e], acc[e], 0, 0, 0);
                }
                p[r] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            }
            if (todo) load_k(b2, phys);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                if (r >= tiles) break;
                if (masked) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int tk = b * kBlockTokens + lg * 4 + j;
                        p[r][j] = tk <= pos[r] && tk >= lo[r] ? p[r][j] : -INFINITY;
                    }
                }
                const float mx = fmaxf(fmaxf(p[r][0], p[r][1]), fmaxf(p[r][2], p[r][3]));
                if (__any(mx > m[r] + kSlackLog2)) {
                    const float mnew = fmaxf(m[r], row_max_4lanes(mx));
                    const float alpha = exp2f(m[r] - (mnew == -INFINITY ? 0.f : mnew));
                    l[r] *= alpha;
#pragma unroll
                    for (int t = 0; t < NU; ++t) o[r][t] *= alpha;
                    m[r] = mnew;
                }
                const float muse = m[r] == -INFINITY ? 0.f : m[r];
#pragma unroll
                for (int j = 0; j < 4; ++j) p[r][j] = exp2f(p[r][j] - muse);
                l[r] += (p[r][0] + p[r][1]) + (p[r][2] + p[r][3]);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int t = 0; t < NU; ++t)
                        o[r][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[t][j], p[r][j], o[r][t], 0, 0, 0);
            }
            if (todo == 0) break;
            load_v(b2, phys);
            at = at2;
            b = b2;
        }
    }

    // merge the four wavefronts' states, one row tile at a time
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        l[r] += __shfl_xor(l[r], 16);
        l[r] += __shfl_xor(l[r], 32);
        if (lg == 0) {
            merge_m[w][r * 16 + l16] = m[r];
            merge_l[w][r * 16 + l16] = l[r];
        }
    }
    __syncthreads();
    float* outp = static_cast<float*>(a.out);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        float M = -INFINITY, L = 0.f;
#pragma unroll
        for (int ww = 0; ww < kAttnWaves; ++ww) M = fmaxf(M, merge_m[ww][r * 16 + l16]);
        const float Muse = M == -INFINITY ? 0.f : M;
#pragma unroll
        for (int ww = 0; ww < kAttnWaves; ++ww)
            L = fmaf(exp2f(merge_m[ww][r * 16 + l16] - Muse), merge_l[ww][r * 16 + l16], L);
        const float f = exp2f(m[r] - Muse);
        if (r > 0) __syncthreads();  // the tile before has been read
#pragma unroll
        for (int t = 0; t < NU; ++t) lds[(w * NU + t) * kWave + lane] = o[r][t] * f;
        __syncthreads();
        const int rr = r0 + r * 16 + l16;
        if (rr < rows_total) {
            const int j = rr / a.group, gh = rr - j * a.group;
            const int64_t hrow = (int64_t)(sg.q0 + j) * a.hq + kvh * a.group + gh;
            const float den = sg.nsplit == 1 ? L + sink_term(a.sinks, kvh * a.group + gh, M) : L;
            const float div = sg.nsplit == 1 ? den : 1.f;
            const int64_t pi = hrow * a.max_splits + s;
            float* dst = sg.nsplit == 1 ? outp + hrow * D : a.part_o + pi * D;
            for (int t = w; t < NU; t += kAttnWaves) {
                f32x4_t O = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ww = 0; ww < kAttnWaves; ++ww) O += lds[(ww * NU + t) * kWave + lane];
                *reinterpret_cast<f32x4u_t*>(dst + t * 16 + lg * 4) = den > 0.f ? O / div : f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
            if (sg.nsplit > 1 && w == 0 && lg == 0)
                *reinterpret_cast<f32x2u_t*>(a.part_ml + 2 * pi) =
                    L > 0.f ? f32x2u_t{M, L} : f32x2u_t{-INFINITY, 0.f};
        }
    }
}

// ------------------------------------------------------------------ MFMA path (bf16)
//
// Persistent, load-balanced schedule.  A unit is one 16-token KV block of one
// (request i, KV head g, row group) pair; units are numbered request by
// request, then head, then row group, then block.  attn_schedule writes the
// per-request unit offsets (a prefix sum over the batch), then attn_persist
// launches a fixed number of workgroups (all resident at once) and gives
// workgroup w the contiguous unit range [U*w/N, U*(w+1)/N), N = min(NWG, U): every
// workgroup streams the same number of KV bytes whatever the context lengths,
// so no workgroup is left running alone at the end.  A pair whose units all
// fall in one range is finished in place; a pair cut by a range boundary
// leaves one partial (normalised output + log-sum-exp) per workgroup in slot
// P + w (P = pair index), and attn_combine_slots merges them.
//
// Launches of short pairs (whole_pairs) skip the schedule: workgroup w walks
// pair w from end to end, and nothing is merged.
//
// Inside a workgroup the NW wavefronts split the pair's query rows (TPW tiles
// of 16 rows each) and share the KV blocks: each block's K and V tiles (16
// tokens x D, contiguous in the paged layout) are copied once, 16 bytes per
// lane, straight from global memory into a ring of NS LDS stages, and read
// from there by every wavefront as MFMA operands.  The load stream runs
// straight across pair boundaries; the ids of the blocks it loads are scalar
// loads issued one step earlier.
//
// The walk goes in steps of two blocks (one where a pair or range ends).  What
// bounds it: with one or two tiles per wavefront, HBM (1.2 GB of a decode
// batch at 5.1 TB/s); with eight tiles per workgroup the chain of a step, its
// LDS time and its scalar instructions.  Two blocks per step halve the
// barriers, waits and maximum tests, double the products in flight, run PV at
// the 32-key rate and make all LDS reads 16 bytes wide and conflict-free; the
// steady-state loop keeps the scalar work of a step at address arithmetic.
// Against one block per step: 43 GB of ragged long contexts 8.70 -> 7.60 ms
// (long-row class 5.96 -> 4.97 ms), 4.6 GB at D = 64 with five tiles 893 ->
// 850 us, a pair of 32 blocks alone on a compute unit 24 -> 14.7 us.
//
// Per 16-row tile, with lane = 16*lg + l16, for a single block:
//   S^T = K Q^T   v_mfma_f32_16x16x32_bf16, A = K (16 keys x 32 dims, lane
//                 holds 8 consecutive dims of key l16: one 16-byte LDS read
//                 of the x-packed K tile), B = Q^T (8 dims of row l16);
//                 the result lane holds keys 4lg..4lg+3 of row l16;
//   O^T += V^T P^T v_mfma_f32_16x16x16_bf16, A = V^T (16 dims x 16 keys, lane
//                 holds 4 keys of dim l16: one 8-byte read of the V^T tile),
//                 B = P^T (the same 4 keys of row l16, straight from the S
//                 registers after the online-softmax update);
// two blocks permute the keys and take the 32-key PV product (see compute).
// The output tile is O^T: lane holds dims 4lg..4lg+3 of row l16, so a row's
// running max and rescale factor live in the lanes that own its scores.
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

typedef short i16x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t as_bf16x8(const uint4& v) { return __builtin_bit_cast(bf16x8_t, v); }


// Scalars of the persistent launch.  The pointers travel as separate
// __restrict__ kernel arguments (MPtrs) so that the compiler can prove the
// metadata arrays are never written by the kernel and read them with scalar
// loads: a vector load there would make every wait on it drain the KV
// prefetch queue.
struct PArgs {
    int num_seqs, hq, hkv, group, max_blocks, num_blocks, window, max_seq_len;
    float scale_log2;
    float inv_scale_log2;  // 1 / scale_log2 (0 when the scale is 0)
    int rows_per_group;   // NW * TPW * 16
    int rg_max;           // row groups per (request, KV head) at most
    int nwg;              // workgroups of the persistent launch
    int spb;              // > 0: fixed number of units per workgroup
    int inline_sched;     // 1: attn_persist computes the unit offsets itself
    int whole;            // 1: workgroup w walks pair w from end to end; no schedule, no slots
    int rows_lo, rows_hi; // the launch's row class: requests whose group * n_i lies in
                          // [rows_lo, rows_hi]; the others belong to another launch
    const float* sinks;   // [Hq] sink logits (natural-log units) or null
};

struct MPtrs {
    const uint16_t* q;
    const uint8_t* kc;
    const uint8_t* vc;
    const int32_t* block_tables;
    const int32_t* seq_lens;
    const int32_t* q_start;
    uint16_t* out;
    int32_t* unit_start;  // [num_seqs + 1] first unit of each request (schedule pass)
    void* slot_o;         // [slots][rows_per_group][D] normalised partial outputs, fp32 or
                          // bf16 (slot_o_index)
    float* slot_lse;      // [slots][rows_per_group]    their log2-sum-exp
    const uint16_t* k_new;  // fused append: [total_q][Hkv][D] new keys, or null
    const uint16_t* v_new;  //               and values
};

struct ReqGeom {
    int q0, n, S, b_lo, nb, rg;
};

// Offset in slot_o of row lr (within the row group), dims d .. d+3 (d % 4 ==
// 0), of slot `slot`.  Each 16-row tile of a slot is stored in the order the
// MFMA output registers hold it: 16-dim column block dt, then lane
// 16 (d / 4 % 4) + lr % 16, then the four dims.
//
// A launch that fills the chip stores the partial outputs in bf16 (the
// log2-sum-exp in fp32), as a split-K merge usually keeps them in the output's
// type: they are normalised, so rounding them adds at most 2^-9 relative error to
// the merged row, and it halves the bytes written at the end of every range and
// read back by the merge.  A launch of few pairs cuts them into fewer ranges than
// would fill the chip, so there are fewer roundings to average out and fewer
// weights that are exactly 1 (one request of 95 blocks, error against 64 bits
// 2.55e-3 with a range per block, 2.75e-3 with 24): its partials stay in fp32
// (2.19e-3; the call 12.7 -> 12.8 us, at most 2 us where 30 pairs have eight
// tiles: 23.7 -> 25.5).
template <int D>
__device__ __forceinline__ int64_t slot_o_index(int64_t slot, int rows_per_group, int lr, int d) {
    const int lane = ((d >> 2) & 3) * 16 + (lr & 15);
    return (slot * rows_per_group + (lr & ~15)) * D + ((d >> 4) * kWave + lane) * 4;
}

// p[k] by a scalar load: p and k are the same in every lane, and no kernel of
// the launch writes the array (constant address space).  Left to itself the
// compiler takes an index carried around a loop as divergent and loads into a
// vector register, whose wait drains the whole prefetch ring.
__device__ __forceinline__ int scalar_load(const int32_t* p, int64_t k) {
    const uint64_t u = (uint64_t)(uintptr_t)(p + k);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(u >> 32));
    typedef const __attribute__((address_space(4))) int32_t* ConstPtr;
    return *(ConstPtr)(uintptr_t)(((uint64_t)hi << 32) | lo);
}

// UNIFORM: i is the same in every lane (scalar loads).
template <bool UNIFORM = false>
__device__ __forceinline__ ReqGeom req_geom(const PArgs& a, const int32_t* __restrict__ q_start,
                                            const int32_t* __restrict__ seq_lens, int i) {
    ReqGeom r;
    r.q0 = UNIFORM ? scalar_load(q_start, i) : q_start[i];
    r.n = (UNIFORM ? scalar_load(q_start, i + 1) : q_start[i + 1]) - r.q0;
    int S = UNIFORM ? scalar_load(seq_lens, i) : seq_lens[i];
    S = max(0, min(S, min(a.max_seq_len, a.max_blocks * kBlockTokens)));
    r.S = S;
    const int key_lo = a.window > 0 ? max(0, S - r.n - a.window + 1) : 0;
    r.b_lo = key_lo / kBlockTokens;
    const int b_hi = (S + kBlockTokens - 1) / kBlockTokens;
    r.nb = max(0, b_hi - r.b_lo);
    const int rows = a.group * max(0, r.n);
    r.rg = min(a.rg_max, (rows + a.rows_per_group - 1) / a.rows_per_group);
    if (rows < a.rows_lo || rows > a.rows_hi) r.rg = 0;  // another launch's request
    return r;
}

// Rows past the launch's reach: a request with more than max_q_len rows can
// need more row groups than the launch provides (rg_max); those rows are not
// computed, and their outputs are written as a quiet NaN instead of being
// left stale.  The calling thread covers requests i0, i0 + step, ... below i1.
template <int D>
__device__ void mark_unreached_rows(const PArgs& a, const int32_t* __restrict__ q_start,
                                    uint16_t* __restrict__ out, int i0, int i1, int step) {
    const int reach = a.rg_max * a.rows_per_group;  // local rows of one (request, KV head)
    for (int i = i0; i < i1; i += step) {
        const int q0 = q_start[i];
        const int rows = a.group * (q_start[i + 1] - q0);
        if (rows < a.rows_lo || rows > a.rows_hi) continue;
        for (int rr = reach; rr < rows; ++rr)
            for (int g = 0; g < a.hkv; ++g) {
                const int64_t hrow = (int64_t)(q0 + rr / a.group) * a.hq + g * a.group + rr % a.group;
                for (int d = 0; d < D; ++d) out[hrow * D + d] = 0x7fc0;  // bf16 quiet NaN
            }
    }
}

// Workgroups that share the U units in equal-share mode: at most one per unit,
// so that every participating workgroup owns at least one unit.
__device__ __forceinline__ int sharing_wgs(const PArgs& a, int U) { return min(a.nwg, max(U, 1)); }

// Workgroup that owns unit u (inverse of the range split).
__device__ __forceinline__ int owner_of(const PArgs& a, int u, int U) {
    if (a.spb > 0) return u / a.spb;
    return (int)(((int64_t)(u + 1) * sharing_wgs(a, U) - 1) / U);
}

// One workgroup: exclusive prefix sum of Hkv * row_groups * blocks over the batch.
template <int D>
__global__ __launch_bounds__(1024) void attn_schedule(PArgs a, const int32_t* __restrict__ q_start,
                                                     const int32_t* __restrict__ seq_lens,
                                                     int32_t* __restrict__ unit_start,
                                                     uint16_t* __restrict__ out) {
    mark_unreached_rows<D>(a, q_start, out, threadIdx.x, a.num_seqs, blockDim.x);
    __shared__ int wsum[16];
    __shared__ int carry_s;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    if (tid == 0) carry_s = 0;
    __syncthreads();
    for (int base = 0; base < a.num_seqs; base += 1024) {
        const int i = base + tid;
        int u = 0;
        if (i < a.num_seqs) {
            const ReqGeom r = req_geom(a, q_start, seq_lens, i);
            u = a.hkv * r.rg * r.nb;
        }
        int x = u;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane == kWave - 1) wsum[wv] = x;
        __syncthreads();
        if (wv == 0) {
            int sv = lane < 16 ? wsum[lane] : 0;
#pragma unroll
            for (int o = 1; o < 16; o <<= 1) {
                const int y = __shfl_up(sv, o);
                if (lane >= o) sv += y;
            }
            if (lane < 16) wsum[lane] = sv;
        }
        __syncthreads();
        const int excl = carry_s + (wv > 0 ? wsum[wv - 1] : 0) + x - u;
        if (i < a.num_seqs) unit_start[i] = excl;
        __syncthreads();
        if (tid == 1023) carry_s = excl + u;
        __syncthreads();
    }
    if (tid == 0) unit_start[a.num_seqs] = carry_s;
}

struct Cursor {
    int i, g, r, b;  // request, KV head, row group, block
    ReqGeom rq;
};

// The pair after (i, g, r), whose request has geometry rq.
__device__ __forceinline__ void next_pair(const PArgs& a, const int32_t* __restrict__ q_start,
                                          const int32_t* __restrict__ seq_lens, int& i, int& g, int& r,
                                          ReqGeom& rq) {
    if (++r < rq.rg) return;
    r = 0;
    if (++g < a.hkv) return;
    g = 0;
    while (++i < a.num_seqs) {
        rq = req_geom<true>(a, q_start, seq_lens, i);
        if (rq.rg > 0 && rq.nb > 0) break;
    }
}

// Batches of at most this many requests are scheduled inside attn_persist:
// every workgroup computes the per-request unit offsets itself (a scan over
// the batch's metadata, cheaper than a separate launch), and workgroup 0
// also stores them for the merge pass.
constexpr int kInlineSchedSeqs = 256;

// Exclusive prefix over the batch of each request's units (Hkv * row groups *
// blocks) into sched[0 .. num_seqs], sched[num_seqs] = total; one wavefront.
__device__ __forceinline__ void sched_prefix(const PArgs& a, const int32_t* __restrict__ q_start,
                                             const int32_t* __restrict__ seq_lens, int32_t* sched,
                                             int lane) {
    int carry = 0;
    for (int base = 0; base < a.num_seqs; base += kWave) {
        const int i = base + lane;
        int u = 0;
        if (i < a.num_seqs) {
            const ReqGeom r = req_geom(a, q_start, seq_lens, i);
            u = a.hkv * r.rg * r.nb;
        }
        int x = u;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (i < a.num_seqs) sched[i] = carry + x - u;
        carry += __shfl(x, kWave - 1);
    }
    if (lane == 0) sched[a.num_seqs] = carry;
}

// Unit range [us, ue) of workgroup w (empty when w has none).
__device__ __forceinline__ void unit_range(const PArgs& a, int U, int w, int& us, int& ue) {
    if (a.spb > 0) {
        us = (int)min((int64_t)U, (int64_t)w * a.spb);
        ue = (int)min((int64_t)U, (int64_t)us + a.spb);
    } else {
        const int n = sharing_wgs(a, U);
        us = w < n ? (int)((int64_t)U * w / n) : U;
        ue = w < n ? (int)((int64_t)U * (w + 1) / n) : U;
    }
}

// Value of a wavefront-uniform load, marked uniform for the compiler (a load
// through LDS or a pointer the kernel also writes is otherwise taken as
// divergent, and so is everything computed from it).
__device__ __forceinline__ int uniform_load(const int32_t* p) { return __builtin_amdgcn_readfirstlane(*p); }

// Cursor of unit u: its request is the largest i with unit_start[i] <= u.
__device__ __forceinline__ Cursor locate_unit(const PArgs& a, const int32_t* __restrict__ q_start,
                                              const int32_t* __restrict__ seq_lens,
                                              const int32_t* unit_start, int u) {
    int lo = 0, hi = a.num_seqs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (uniform_load(unit_start + mid) <= u) lo = mid; else hi = mid - 1;
    }
    Cursor c;
    c.i = lo;
    c.rq = req_geom<true>(a, q_start, seq_lens, lo);
    const int off = u - uniform_load(unit_start + lo);
    const int pq = off / c.rq.nb;  // pair within the request: head * rg + row group
    c.g = pq / c.rq.rg;
    c.r = pq - c.g * c.rq.rg;
    c.b = c.rq.b_lo + (off - pq * c.rq.nb);
    return c;
}

// One online-softmax step of a 16-row tile over NB consecutive 16-key blocks.
// sacc holds raw scores <q, k> in the MFMA result layout (lane 16 lg + l16:
// keys key0 .. key0 + 3 of each block for the tile's row l16, key0 = 16 b + 4 lg
// in the first); row_j is the
// row's draft position (-1: no row) and p_first the position of the request's
// first row.  The exponentials are taken against the stored maximum m as long
// as no score exceeds it by more than 2^kSlackLog2; only then (on a row's
// first keys, and rarely after) does the wavefront reduce the new row maximum
// over the row's four lanes and rescale l and o.  The weights stay below
// 2^kSlackLog2, and bf16 rounds them with the same relative error at any
// magnitude.  pw receives the weights as the bf16 B operand of the PV product,
// two words per block.
template <int NB, int DT>
__device__ __forceinline__ void softmax_step(const f32x4_t (&sacc)[NB], bool need_mask, int row_j,
                                             int p_first, const int (&key0)[NB], int window, float c,
                                             float inv_c, float& m, float& l, float& thr, float& neg_m,
                                             f32x4_t (&o)[DT], uint32_t (&pw)[2 * NB]) {
    float sv[4 * NB];
#pragma unroll
    for (int r = 0; r < 4 * NB; ++r) sv[r] = sacc[r / 4][r % 4];
    if (need_mask) {
        const int p = p_first + row_j;
#pragma unroll
        for (int r = 0; r < 4 * NB; ++r) {
            const int key = key0[r / 4] + r % 4;
            const bool vis = row_j >= 0 && key <= p && (window == 0 || key > p - window);
            sv[r] = vis ? sv[r] : -INFINITY;
        }
    }
    float mx = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
    if constexpr (NB == 2) mx = fmaxf(mx, fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
    if (__builtin_amdgcn_ballot_w64(!(mx <= thr))) {
        const float rmax = row_max_4lanes(mx) * c;
        if (rmax > m) {
            // m = -inf: nothing accumulated yet, alpha = 0 keeps it 0
            const float alpha = __builtin_amdgcn_exp2f(m - rmax);
            l *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[dt] *= alpha;
            m = rmax;
            neg_m = -rmax;
            thr = (rmax + kSlackLog2) * inv_c;
        }
    }
    // exponent arguments are <= kSlackLog2: the raw v_exp_f32 is exact enough
    // and results below 2^-126 only flush to zero
    float pr[4 * NB];
#pragma unroll
    for (int r = 0; r < 4 * NB; ++r) pr[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[r], c, neg_m));
#pragma unroll
    for (int h = 0; h < NB; ++h) {
        l += (pr[4 * h] + pr[4 * h + 1]) + (pr[4 * h + 2] + pr[4 * h + 3]);
        pw[2 * h] = pack_bf16x2(pr[4 * h], pr[4 * h + 1]);
        pw[2 * h + 1] = pack_bf16x2(pr[4 * h + 2], pr[4 * h + 3]);
    }
}

// Wait until at most n blocks' loads (CPT per thread each, n <= MAXN) are in
// flight.  n is wavefront-uniform; STEADY, its value in the steady state, is
// tested first.
template <int CPT, int STEADY, int MAXN>
__device__ __forceinline__ void wait_blocks(int n) {
    if constexpr (STEADY >= 0) {
        if (n == STEADY) wait_vmcnt<CPT * STEADY>();
        else wait_blocks<CPT, -1, MAXN>(n);
    } else if constexpr (MAXN == 0) {
        wait_vmcnt<0>();
    } else {
        if (n >= MAXN) wait_vmcnt<CPT * MAXN>();
        else wait_blocks<CPT, -1, MAXN - 1>(n);
    }
}

// Global->LDS loads need about sixteen wavefronts per compute unit to reach
// full HBM bandwidth, so one-tile configurations are held to four waves per
// SIMD (at most 128 registers each).
// Waves per SIMD the persistent kernel is built for.  The four-wavefront
// two-tile kernels are held to three (168 registers): three workgroups per
// compute unit hide a step's chain of LDS reads, products and exponentials
// better than two with deeper rings (long-row class of the 43 GB batch 4.97
// against 5.06 ms).  The fused append's then keeps some values in scratch (and so
// does its five-tile kernel at 256 registers), reloaded on pair switches, patched
// blocks and in the steps between them and the steady state, which holds none.
template <int TPW, int NW>
constexpr int persist_waves_per_eu() { return TPW == 1 ? 4 : (NW == 4 && TPW == 2 ? 3 : 2); }

// APPEND: the fused KV append (verify_attention_append).  The request's new
// tokens, positions S_i - n_i .. S_i - 1 of rows q_start[i] .. q_start[i+1]-1,
// are taken from k_new / v_new: after a block holding some of them has landed
// in LDS, the workgroup overwrites their K and V there (one extra barrier, on
// those blocks only), and the workgroup of the pair's first row group also
// stores them into the cache.  Readers never depend on that store, so no
// ordering between workgroups is needed.
//
// Slot: the type of the partial outputs (uint16_t: bf16, or float; slot_o_index).
template <int D, int NW, int TPW, int NS, bool APPEND, typename Slot>
__global__ __launch_bounds__(NW * kWave)
__attribute__((amdgpu_waves_per_eu(persist_waves_per_eu<TPW, NW>()))) void attn_persist(
    PArgs a, const uint16_t* __restrict__ qg, const uint8_t* __restrict__ kcg,
    const uint8_t* __restrict__ vcg, const int32_t* __restrict__ block_tables,
    const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ q_start,
    int32_t* __restrict__ unit_start, uint16_t* __restrict__ out,
    Slot* __restrict__ slot_o, float* __restrict__ slot_lse,
    const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new) {
    constexpr int NT = NW * kWave;
    constexpr int TILE_BYTES = kBlockTokens * D * 2;  // one (block, head) K or V tile
    constexpr int CH = 2 * TILE_BYTES / 16;           // 16-byte chunks per block (K then V)
    constexpr int CPT = CH / NT;                      // chunks per thread per block
    constexpr int KC = D / 32;                        // QK^T steps of 32 dims
    constexpr int DT = D / 16;                        // PV output tiles of 16 dims
    constexpr int ROWS = NW * TPW * 16;
    constexpr int STEP = 2;                           // blocks per step at most
    static_assert(CH % NT == 0, "every thread loads the same number of chunks");
    static_assert(NS >= 4 && NS <= 32 && CPT * (NS - 1) < 64, "ok_mask bits and vmcnt range");
    static_assert(2 * TILE_BYTES >= (int)sizeof(int32_t) * (kInlineSchedSeqs + 1), "schedule scan in a stage");

    __shared__ __attribute__((aligned(16))) uint8_t stage[NS][2 * TILE_BYTES];
    // the schedule scan lives in the last stage, which is first loaded after
    // the first step's barrier
    int32_t* const sched = reinterpret_cast<int32_t*>(stage[NS - 1]);

    const int w = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane(tid / kWave);  // wavefront-uniform
    const int l16 = lane & 15, lg = lane >> 4;

    int us, ue;
    Cursor c0;
    if (a.whole) {
        // one pair per workgroup, unit u of it is block b_lo + u
        const int per_req = a.hkv * a.rg_max;
        c0.i = w / per_req;
        c0.g = (w - c0.i * per_req) / a.rg_max;
        c0.r = w - c0.i * per_req - c0.g * a.rg_max;
        c0.rq = req_geom<true>(a, q_start, seq_lens, c0.i);
        c0.b = c0.rq.b_lo;
        if (c0.g == 0 && c0.r == 0 && tid == 0)
            mark_unreached_rows<D>(a, q_start, out, c0.i, c0.i + 1, 1);
        if (c0.r >= c0.rq.rg) return;
        us = 0;
        ue = c0.rq.nb;
        if (ue == 0) {  // no key: zeros for the pair's rows
            const int r1 = min(ROWS, a.group * c0.rq.n - c0.r * ROWS);
            for (int e = tid; e < r1 * (D / 4); e += NT) {
                const int rr = c0.r * ROWS + e / (D / 4);
                const int64_t hrow =
                    (int64_t)(c0.rq.q0 + rr / a.group) * a.hq + c0.g * a.group + rr % a.group;
                *reinterpret_cast<uint2*>(out + hrow * D + e % (D / 4) * 4) = make_uint2(0, 0);
            }
            return;
        }
    } else {
        const int32_t* ustart = unit_start;
        if (a.inline_sched) {
            if (wv == 0) {
                sched_prefix(a, q_start, seq_lens, sched, lane);
                if (w == 0) {
                    for (int i = lane; i <= a.num_seqs; i += kWave) unit_start[i] = sched[i];
                    mark_unreached_rows<D>(a, q_start, out, lane, a.num_seqs, kWave);
                }
            }
            __syncthreads();
            ustart = sched;
        }
        const int U = uniform_load(ustart + a.num_seqs);
        unit_range(a, U, w, us, ue);
        if (us >= ue) return;
        c0 = locate_unit(a, q_start, seq_lens, ustart, us);
    }

    const uint32_t stage_lds =
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)&stage[0][0];
    // One unit = one block's K and V tiles, copied into an LDS stage with CPT
    // global->LDS loads of 1 KiB per wavefront: wavefront w copies chunks
    // [w CPT, (w + 1) CPT) of the 2 TILE_BYTES / 1 KiB (K's first).  A
    // wavefront's loads from one tile share m0, the scalar base address and
    // the lane offset; the instruction's immediate offset, which the hardware
    // adds to both the global and the LDS address, steps through them.  Every
    // call issues exactly CPT loads, invalid block ids reading block 0
    // (compute skips them through ok_mask), so the explicit vmcnt waits below
    // count exactly.
    // Bit s: stage s holds a valid block.  Every wavefront runs the same
    // loader steps, so each keeps its own copy in a scalar register.
    uint32_t ok_mask = 0;
    const uint32_t lane16 = (uint32_t)lane * 16;
    constexpr int TILE_LOADS = TILE_BYTES / 1024;         // loads of one tile
    constexpr int RUN = CPT < TILE_LOADS ? CPT : TILE_LOADS;  // of them by one wavefront
    auto dma_unit = [&](int g, int st, int phys) {
        const bool ok = phys >= 0 && phys < a.num_blocks;
        ok_mask = ok ? (ok_mask | (1u << st)) : (ok_mask & ~(1u << st));
        phys = ok ? phys : 0;
        const int64_t off = ((int64_t)phys * a.hkv + g) * TILE_BYTES;
        const uint32_t base = stage_lds + st * (2 * TILE_BYTES);
#pragma unroll
        for (int c = 0; c < CPT; c += RUN) {
            const int first = wv * CPT + c;  // this run's first load of the block's 2 TILE_LOADS
            const uint8_t* src = first < TILE_LOADS ? kcg + off + first * 1024
                                                    : vcg + off + (first - TILE_LOADS) * 1024;
            dma16_run<RUN>(base + first * 1024, src, lane16);
        }
    };

    // ---- state of the pair being computed: the pair cc points into
    Cursor cc = c0;
    int st_ps = 0;  // first unit of the pair
    bool active = false;
    bf16x8_t qop[TPW][KC];
    int row_j[TPW];
    f32x4_t o[TPW][DT];
    // Online softmax state per tile, in the log2 domain: m_r is the maximum
    // the row's exponentials are taken against (identical in the four lanes
    // that hold the row), thr the raw score above which a lane needs a new
    // maximum, neg_m = -m_r (0 while the row has seen no key).  With five tiles
    // m_r is taken from the other two where it is needed (rarely): its five
    // registers, and five of sink logits that are now read when a pair is done,
    // are what kept that kernel from fitting 256 (1024 pairs of 64 blocks at head
    // dim 64: walk 62.6 -> 59.2 us).
    constexpr bool KEEP_M = TPW < 5;
    float m_kept[TPW], l_r[TPW], thr[TPW], neg_m[TPW];
    auto m_r = [&](int t) { return KEEP_M ? m_kept[t] : thr[t] == -INFINITY ? -INFINITY : -neg_m[t]; };
    // APPEND: the pair's new-token positions [st_nlo, st_nhi) (those the walk
    // reaches) and the position of its first row, S_i - n_i
    int st_nlo = 0, st_nhi = 0, st_p0 = 0;

    // The pair of cc, reached at unit u.
    auto init_pair = [&](int u) {
        st_ps = u - (cc.b - cc.rq.b_lo);
        if constexpr (APPEND) {
            const int s_raw = scalar_load(seq_lens, cc.i);
            st_p0 = s_raw - cc.rq.n;
            st_nlo = max(st_p0, 0);
            st_nhi = min(s_raw, cc.rq.S);
        }
        const int rows = a.group * cc.rq.n;
        const int wrow0 = cc.r * ROWS + wv * TPW * 16;
        active = wrow0 < rows;
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            const int rr = wrow0 + t * 16 + l16;
            const bool valid = rr < rows;
            const int j = rr / a.group, gh = rr - j * a.group;
            row_j[t] = valid ? j : -1;
            const int64_t base = ((int64_t)(cc.rq.q0 + j) * a.hq + cc.g * a.group + gh) * D;
#pragma unroll
            for (int cc = 0; cc < KC; ++cc) {
                uint4 v = make_uint4(0, 0, 0, 0);
                if (valid) v = ld16(qg + base + (cc * 4 + lg) * 8);
                qop[t][cc] = as_bf16x8(v);
            }
            m_kept[t] = -INFINITY;
            l_r[t] = 0.f;
            thr[t] = -INFINITY;
            neg_m[t] = 0.f;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) o[t][dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        }
        // Settle the Q loads here, on the (rare) pair-switch path.  Otherwise
        // the compiler cannot tell whether they are still in flight when the
        // next block's MFMA reads the operands, and waits for the whole load
        // queue, prefetched KV blocks included, before every block.
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    };

    auto flush_pair = [&]() {
        if (!active) return;
        const bool whole = st_ps >= us && st_ps + cc.rq.nb <= ue;
        const int rows = a.group * cc.rq.n;
        const int64_t slot = (int64_t)(cc.i * a.hkv + cc.g) * a.rg_max + cc.r + w;
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            float L = l_r[t];
            L += __shfl_xor(L, 16);
            L += __shfl_xor(L, 32);
            const int lr = (wv * TPW + t) * 16 + l16;
            const int rr = cc.r * ROWS + lr;
            if (rr >= rows) continue;
            if (whole) {
                const int j = rr / a.group, gh = rr - j * a.group;
                const float den = L + sink_term(a.sinks, cc.g * a.group + gh, m_r(t));
                const float inv = den > 0.f ? 1.f / den : 0.f;
                const int64_t hrow = (int64_t)(cc.rq.q0 + j) * a.hq + cc.g * a.group + gh;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    const int d0 = dt * 16 + 4 * lg;
                    const uint2 v = make_uint2(pack_bf16x2(o[t][dt][0] * inv, o[t][dt][1] * inv),
                                               pack_bf16x2(o[t][dt][2] * inv, o[t][dt][3] * inv));
                    *reinterpret_cast<uint2*>(out + hrow * D + d0) = v;
                }
            } else {
                // the tile's 16 rows x D values in register order (see
                // slot_o_index): each store writes 512 bytes (fp32: 1 KiB) contiguous
                const float inv = L > 0.f ? 1.f / L : 0.f;
                const int64_t srow = slot * ROWS + lr;
                Slot* tb = slot_o + (slot * ROWS + (wv * TPW + t) * 16) * D + lane * 4;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    if constexpr (sizeof(Slot) == 4)
                        *reinterpret_cast<f32x4u_t*>(tb + dt * (kWave * 4)) = o[t][dt] * inv;
                    else
                        *reinterpret_cast<uint2*>(tb + dt * (kWave * 4)) =
                            make_uint2(pack_bf16x2(o[t][dt][0] * inv, o[t][dt][1] * inv),
                                       pack_bf16x2(o[t][dt][2] * inv, o[t][dt][3] * inv));
                }
                if (lg == 0) slot_lse[srow] = L > 0.f ? m_r(t) + log2f(L) : -INFINITY;
            }
        }
    };

    // One step of the walk: block b in stage st, and with NB = 2 block b + 1
    // in stage st2.
    //
    // Two blocks are one 32-key step.  The PV product then takes 32 keys per
    // MFMA, and the key order is chosen so that every LDS read is 16 bytes
    // wide and free of bank conflicts: row m of the two QK products stands for
    // the keys below (t within the block), so that lane group lg ends up with
    // eight consecutive keys of one block, the 16 bytes of a V^T row that it
    // reads as its share of the PV operand.
    //     m        0-3     4-7      8-11    12-15
    //     first    A 0-3   A 8-11   B 4-7   B 12-15
    //     second   A 4-7   A 12-15  B 0-3   B 8-11
    // (Single blocks read V^T by 8 bytes, with two-way conflicts: the two
    // 8-byte halves of a row lie in the same bank group as those of the row
    // eight further on.)
    auto compute = [&](auto nb, bool masked, int st, int st2, int b) {
        constexpr int NB = decltype(nb)::value;
        const bool b_row = NB == 2 && l16 >= 8, b_lane = NB == 2 && lg >= 2;
        const uint8_t* const kb = stage[b_row ? st2 : st] + lg * 256;
        const uint8_t* const vb = stage[b_lane ? st2 : st] + TILE_BYTES;
        int kt[NB];  // byte offset of this lane's key in each QK product
        if constexpr (NB == 2) {
            kt[0] = (((l16 >> 2) & 1) * 8 + (l16 >> 3) * 4 + (l16 & 3)) * 16;
            kt[1] = kt[0] ^ 64;
        } else {
            kt[0] = l16 * 16;
        }
        f32x4_t sacc[TPW][NB];
#pragma unroll
        for (int t = 0; t < TPW; ++t)
#pragma unroll
            for (int h = 0; h < NB; ++h) sacc[t][h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int cc4 = 0; cc4 < KC; ++cc4) {
#pragma unroll
            for (int h = 0; h < NB; ++h) {
                const bf16x8_t kop = as_bf16x8(*reinterpret_cast<const uint4*>(kb + kt[h] + cc4 * 1024));
#pragma unroll
                for (int t = 0; t < TPW; ++t)
                    sacc[t][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop, qop[t][cc4], sacc[t][h], 0, 0, 0);
            }
        }
        const int p_first = cc.rq.S - cc.rq.n;  // position of the request's first query row
        int key0[NB];
        if constexpr (NB == 2) {
            const int k8 = (b + b_lane) * kBlockTokens + (lg & 1) * 8;
            key0[0] = k8 + (b_lane ? 4 : 0);
            key0[1] = k8 + (b_lane ? 0 : 4);
        } else {
            key0[0] = b * kBlockTokens + 4 * lg;
        }
        uint32_t pw[TPW][2 * NB];
#pragma unroll
        for (int t = 0; t < TPW; ++t) {
            float m = m_r(t);
            softmax_step<NB, DT>(sacc[t], masked, row_j[t], p_first, key0, a.window, a.scale_log2,
                                 a.inv_scale_log2, m, l_r[t], thr[t], neg_m[t], o[t], pw[t]);
            m_kept[t] = m;
            if constexpr (NB == 2) {  // ascending keys
                const uint32_t w0 = pw[t][0], w1 = pw[t][1];
                pw[t][0] = b_lane ? pw[t][2] : w0;
                pw[t][1] = b_lane ? pw[t][3] : w1;
                pw[t][2] = b_lane ? w0 : pw[t][2];
                pw[t][3] = b_lane ? w1 : pw[t][3];
            }
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
            if constexpr (NB == 2) {
                const bf16x8_t vop = as_bf16x8(
                    *reinterpret_cast<const uint4*>(vb + (dt * 16 + l16) * 32 + (lg & 1) * 16));
#pragma unroll
                for (int t = 0; t < TPW; ++t)
                    o[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        vop, as_bf16x8(make_uint4(pw[t][0], pw[t][1], pw[t][2], pw[t][3])), o[t][dt], 0, 0, 0);
            } else {
                const i16x4_t vop = __builtin_bit_cast(
                    i16x4_t, *reinterpret_cast<const uint2*>(vb + (dt * 16 + l16) * 32 + lg * 8));
#pragma unroll
                for (int t = 0; t < TPW; ++t)
                    o[t][dt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                        vop, __builtin_bit_cast(i16x4_t, make_uint2(pw[t][0], pw[t][1])), o[t][dt], 0, 0, 0);
            }
        }
    };
    // The blocks of a step whose ids are valid.
    auto compute_step = [&](bool masked, int st, int st2, bool two, int b) {
        const bool ok1 = (ok_mask >> st) & 1u, ok2 = two && ((ok_mask >> st2) & 1u);
        // two plain ifs: with an else the compiler keeps the accumulators twice
        const bool both = ok1 && ok2 && active, one = (ok1 || ok2) && !both && active;
        if (both) compute(std::integral_constant<int, 2>{}, masked, st, st2, b);
        if (one) compute(std::integral_constant<int, 1>{}, masked, ok1 ? st : st2, 0, ok1 ? b : b + 1);
    };

    // APPEND: overwrite the new tokens of block b in stage st with their K and
    // V from k_new / v_new (16 bytes = 8 dims of one token per step), and, in
    // the pair's first row group, store them into the cache block as well.
    auto patch_new = [&](int st, int b) {
        constexpr int DC = D / 8;  // 16-byte chunks per key
        const int pos0 = b * kBlockTokens;
        const int t_lo = max(st_nlo - pos0, 0), t_hi = min(st_nhi - pos0, kBlockTokens);
        uint8_t* ks = stage[st];
        uint16_t* vs = reinterpret_cast<uint16_t*>(stage[st] + TILE_BYTES);
        const bool writer = cc.r == 0;
        const int phys = scalar_load(block_tables, (int64_t)cc.i * a.max_blocks + b);
        const int64_t toff = ((int64_t)phys * a.hkv + cc.g) * TILE_BYTES;
        uint8_t* kw = const_cast<uint8_t*>(kcg) + toff;
        uint16_t* vw = reinterpret_cast<uint16_t*>(const_cast<uint8_t*>(vcg) + toff);
        // K and V of one token's 8 dims per step, both loads in flight together
        for (int e = tid; e < (t_hi - t_lo) * DC; e += NT) {
            const int t = t_lo + e / DC, dc = e % DC;
            const int64_t row = cc.rq.q0 + (pos0 + t - st_p0);
            const int64_t src = (row * a.hkv + cc.g) * D + dc * 8;
            const uint4 kv = ld16(k_new + src);
            const uint4 vv = ld16(v_new + src);
            const int kchunk = dc * kBlockTokens + t;
            *reinterpret_cast<uint4*>(ks + kchunk * 16) = kv;
            const uint32_t vh[4] = {vv.x, vv.y, vv.z, vv.w};
#pragma unroll
            for (int k = 0; k < 8; ++k)
                vs[(dc * 8 + k) * kBlockTokens + t] = (uint16_t)(vh[k >> 1] >> (16 * (k & 1)));
            if (writer) {
                *reinterpret_cast<uint4*>(kw + kchunk * 16) = kv;
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    vw[(dc * 8 + k) * kBlockTokens + t] = (uint16_t)(vh[k >> 1] >> (16 * (k & 1)));
            }
        }
    };

    // ---- pipeline: a ring of NS LDS stages, one block each, in walk order.  A
    // step computes the next two blocks, or one where the pair or the range
    // ends after it: wait for this thread's loads of the step's blocks (younger
    // ones may stay in flight), barrier (everyone's loads of them have landed
    // and everyone is done with the blocks before), refill the stages of the
    // previous step, compute.  `issued` and `done` count blocks from us.
    const int total = ue - us;
    int issued = 0, done = 0;
    // The loader's next two blocks (head, block id): `fetched` blocks have been
    // looked up, the l_ values are the cursor of the next, whose request's table
    // row starts at lrow.  The ids are scalar loads, issued once a step's
    // compute has read its LDS operands (so that no LDS wait there also waits
    // for them) and consumed after the next barrier.
    int l_i = c0.i, l_g = c0.g, l_rg = c0.r, l_b = c0.b, l_end = c0.rq.b_lo + c0.rq.nb;
    const int32_t* lrow = block_tables + (int64_t)l_i * a.max_blocks;
    int fetched = 0, g0 = 0, g1 = 0, phys0 = 0, phys1 = 0;
    auto fetch_to = [&](int want) {  // look up blocks until `want` are (at most two ahead)
        if (fetched + 2 == want && l_b + 2 < l_end) {
            g0 = g1 = l_g;
            phys0 = scalar_load(lrow, l_b);
            phys1 = scalar_load(lrow, l_b + 1);
            l_b += 2;
            fetched = want;
            return;
        }
#pragma unroll 1
        while (fetched < want) {
            g0 = g1;
            phys0 = phys1;
            g1 = l_g;
            phys1 = scalar_load(lrow, l_b);
            ++fetched;
            if (++l_b == l_end && fetched < total) {
                ReqGeom rq = req_geom<true>(a, q_start, seq_lens, l_i);  // rather than kept
                next_pair(a, q_start, seq_lens, l_i, l_g, l_rg, rq);
                l_b = rq.b_lo;
                l_end = rq.b_lo + rq.nb;
                lrow = block_tables + (int64_t)l_i * a.max_blocks;
            }
        }
        if (want == total && fetched == issued + 1) {  // the last block
            g0 = g1;
            phys0 = phys1;
        }
    };
    int st_next = 0;  // stage of the next block to load
    auto issue_to = [&](int want) {  // load blocks until `want` are (at most two)
#pragma unroll 1
        while (issued < want) {
            dma_unit(g0, st_next, phys0);
            st_next = st_next == NS - 1 ? 0 : st_next + 1;
            g0 = g1;
            phys0 = phys1;
            ++issued;
        }
    };
#pragma unroll 1
    while (issued < min(NS - 1, total)) {
        fetch_to(min(issued + 2, total));
        issue_to(min(min(issued + 2, NS - 1), total));
    }
    fetch_to(min(issued + 2, total));

    int st = 0;
    bool fresh = true;
    for (;;) {
        if (fresh) init_pair(us + done);
        fresh = false;
        const int p_first = cc.rq.S - cc.rq.n;
        // Steady state: steps whose blocks every row sees in full, with as
        // many blocks to load, and no pair end for the walk or the loader.
        // Nothing is left to decide in them but the ids' validity: the scalar
        // work per block, which all wavefronts repeat, was as long as the
        // products' (94 scalar against 98 vector instructions per block).
        {
            int lim = min(cc.rq.b_lo + cc.rq.nb, (p_first + 1) >> 4) - cc.b;
            if constexpr (APPEND) lim = min(lim, (st_nlo >> 4) - cc.b);
            lim = min(min(lim, total - fetched), l_end - 1 - l_b);
            if (a.window > 0 && cc.b * kBlockTokens < cc.rq.S - a.window) lim = 0;
            if (issued - done != NS - STEP || g0 != l_g || g1 != l_g) lim = 0;
            const int steps = __builtin_amdgcn_readfirstlane(lim >= STEP ? lim / STEP : 0);
            if (steps > 0) {
                const int32_t* ids = lrow + l_b;
#pragma unroll 1
                for (int k = 0; k < steps; ++k) {
                    wait_vmcnt<CPT * (NS - 2 * STEP)>();
                    lds_barrier();
                    dma_unit(l_g, st_next, phys0);
                    st_next = st_next == NS - 1 ? 0 : st_next + 1;
                    dma_unit(l_g, st_next, phys1);
                    st_next = st_next == NS - 1 ? 0 : st_next + 1;
                    const int st2 = st == NS - 1 ? 0 : st + 1;
                    compute_step(false, st, st2, true, cc.b);
                    asm volatile("" ::: "memory");
                    phys0 = scalar_load(ids, 0);
                    phys1 = scalar_load(ids, 1);
                    ids += STEP;
                    st = st2 == NS - 1 ? 0 : st2 + 1;
                }
                issued += steps * STEP;
                done += steps * STEP;
                fetched += steps * STEP;
                l_b += steps * STEP;
                cc.b += steps * STEP;
            }
        }
        const int left = cc.rq.b_lo + cc.rq.nb - cc.b;  // blocks of the pair from here
        if (left > 0 && done < total) {
            const bool two = left > 1 && done + 1 < total;
            const int cnt = two ? 2 : 1;
            const int st2 = st == NS - 1 ? 0 : st + 1;
            wait_blocks<CPT, NS - 2 * STEP, NS - 2>(issued - done - cnt);
            lds_barrier();
            issue_to(min(done + NS, total));
            if constexpr (APPEND) {
                // block-uniform: every wavefront takes the same branches
                const int pos0 = cc.b * kBlockTokens;
                if (pos0 < st_nhi && pos0 + cnt * kBlockTokens > st_nlo) {
#pragma unroll 1
                    for (int h = 0; h < cnt; ++h) {
                        const int pos = pos0 + h * kBlockTokens, sth = h ? st2 : st;
                        if (((ok_mask >> sth) & 1u) && pos < st_nhi && pos + kBlockTokens > st_nlo)
                            patch_new(sth, cc.b + h);
                    }
                    lds_barrier();
                }
            }
            const bool masked = block_needs_mask(cc.b, p_first, cc.rq.S, a.window) ||
                                (two && block_needs_mask(cc.b + 1, p_first, cc.rq.S, a.window));
            compute_step(masked, st, st2, two, cc.b);
            asm volatile("" ::: "memory");
            fetch_to(min(issued + 2, total));
            done += cnt;
            cc.b += cnt;
            st = two ? (st2 == NS - 1 ? 0 : st2 + 1) : st2;
            if (left > cnt && done < total) continue;
        }
        flush_pair();
        if (done >= total) return;
        next_pair(a, q_start, seq_lens, cc.i, cc.g, cc.r, cc.rq);
        cc.b = cc.rq.b_lo;
        fresh = true;
    }
}

// Merges the partial slots of pairs cut by workgroup range boundaries, and
// writes the zero output of rows whose request has no key.  Grid (pairs, row
// chunks); a thread owns one row and four consecutive output dimensions.  The
// slots of a row are read kCombineSlots at a time, every load of a round
// issued before any is used, and merged with a running maximum.  In a full
// batch a pair is cut into a handful of slots and one round covers it.  Where
// few pairs are cut into many (SG = 4), four thread groups share a row: each
// takes every fourth round, and their sums are merged through LDS (24 slots:
// three rounds of latency -> one; one request of 95 blocks, whole call 16.3 ->
// 13.1 us).  Eight wavefronts per SIMD hide a round's latency; the partials stay
// packed until they are added, which is what lets a round fit the 64 registers
// that leaves (unpacked at once they went to scratch; one request 13.1 -> 12.6 us,
// 512 pairs of up to 120 blocks and 4 rows 20.5 -> 19.4).
constexpr int kCombineThreads = 256;
constexpr int kCombineSlots = 8;

// The four partial values of a slot, as they are stored: bf16 pairs, or fp32.
__device__ __forceinline__ f32x4_t unpack4(const uint2& v) {
    return f32x4_t{bf16_lo(v.x), bf16_hi(v.x), bf16_lo(v.y), bf16_hi(v.y)};
}
__device__ __forceinline__ f32x4_t unpack4(const f32x4_t& v) { return v; }

// Slot: the type of the partial outputs, as in attn_persist.
template <int D, int SG, typename Slot>
__global__ __launch_bounds__(kCombineThreads) __attribute__((amdgpu_waves_per_eu(sizeof(Slot) == 2 ? 8 : 5)))
void attn_combine_slots(
    PArgs a, const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ q_start,
    const int32_t* __restrict__ unit_start, const Slot* __restrict__ slot_o,
    const float* __restrict__ slot_lse, uint16_t* __restrict__ out) {
    using Four = std::conditional_t<sizeof(Slot) == 2, uint2, f32x4u_t>;  // four partial values
    constexpr int QUADS = D / 4;                       // 4-dim vectors per row
    constexpr int RPB = kCombineThreads / QUADS / SG;  // rows per workgroup
    const int P = blockIdx.x;
    const int per_req = a.hkv * a.rg_max;
    const int i = P / per_req;
    const int rem = P - i * per_req;
    const int g = rem / a.rg_max, rg = rem - g * a.rg_max;
    // the request's metadata and unit offsets are read together, before any
    // test, so that they cost one memory latency instead of one each
    const int U = unit_start[a.num_seqs];
    const int ustart_i = unit_start[i];
    const ReqGeom rq = req_geom(a, q_start, seq_lens, i);
    if (rg >= rq.rg) return;
    const int ROWS = a.rows_per_group;
    const int group_rows = min(ROWS, a.group * rq.n - rg * ROWS);  // rows of this row group
    if ((int)blockIdx.y * RPB >= group_rows) return;  // before the divisions of owner_of
    const bool empty = rq.nb == 0;
    int wf = 0, wl = 0;
    if (!empty) {
        const int ps = ustart_i + (g * rq.rg + rg) * rq.nb;
        wf = owner_of(a, ps, U);
        wl = owner_of(a, ps + rq.nb - 1, U);
        if (wf == wl) return;  // finished in place by its only workgroup
    }
    const int item = threadIdx.x % (kCombineThreads / SG);   // (row, quad) of the workgroup
    const int sg = threadIdx.x / (kCombineThreads / SG);     // slot group
    const int d0 = (item % QUADS) * 4;
    // one pass, unless the request has more rows than the launch was sized for
    for (int base = blockIdx.y * RPB; base < group_rows; base += gridDim.y * RPB) {
        const int lr = base + item / QUADS;  // row within the group
        const int rr = rg * ROWS + lr;
        const bool in_row = lr < group_rows;
        f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
        float M = -INFINITY, L = 0.f;
        if (!empty && in_row) {
            // slots of the pair: one per workgroup wf .. wl; a slot holding
            // log-sum-exp -inf (no visible key in its range) adds nothing
            const int64_t slot0 = (int64_t)P + wf;
            const int ns = wl - wf + 1;
            for (int s0 = sg * kCombineSlots; s0 < ns; s0 += SG * kCombineSlots) {
                // every load is issued unconditionally (slots past the pair's last
                // re-read the last one and are masked afterwards), so that the
                // round's loads leave back to back; conditional loads compiled to a
                // branch and a wait per slot, one memory latency each
                float lse[kCombineSlots];
                Four v[kCombineSlots];
#pragma unroll
                for (int k = 0; k < kCombineSlots; ++k) {
                    const int64_t sl = slot0 + min(s0 + k, ns - 1);
                    lse[k] = slot_lse[sl * ROWS + lr];
                    v[k] = *reinterpret_cast<const Four*>(slot_o + slot_o_index<D>(sl, ROWS, lr, d0));
                }
#pragma unroll
                for (int k = 0; k < kCombineSlots; ++k) {
                    const bool in = s0 + k < ns;
                    lse[k] = in ? lse[k] : -INFINITY;
                    v[k] = in ? v[k] : Four{};
                }
                float m = M;
#pragma unroll
                for (int k = 0; k < kCombineSlots; ++k) m = fmaxf(m, lse[k]);
                // without a branch for m = -inf, below which the compiler would
                // move the loads of the values, a second memory latency per round
                const float mu = m == -INFINITY ? 0.f : m;
                // rescale what earlier rounds summed (nothing yet: M = -inf gives 0)
                const float r = __builtin_amdgcn_exp2f(M - mu);
                L *= r;
                acc *= r;
#pragma unroll
                for (int k = 0; k < kCombineSlots; ++k) {
                    const float f = __builtin_amdgcn_exp2f(lse[k] - mu);
                    L += f;
                    acc += f * unpack4(v[k]);
                }
                M = m;
            }
        }
        if constexpr (SG > 1) {
            // slot groups 1 .. SG - 1 hand their sums to group 0, which merges
            // them in ascending order
            __shared__ float sm[SG][2][kCombineThreads / SG];
            __shared__ f32x4_t so[SG][kCombineThreads / SG];
            sm[sg][0][item] = M;
            sm[sg][1][item] = L;
            so[sg][item] = acc;
            __syncthreads();
            if (sg == 0) {
                float m = M;
#pragma unroll
                for (int k = 1; k < SG; ++k) m = fmaxf(m, sm[k][0][item]);
                if (m != -INFINITY) {
                    const float r = __builtin_amdgcn_exp2f(M - m);
                    L *= r;
                    acc *= r;
#pragma unroll
                    for (int k = 1; k < SG; ++k) {
                        const float f = __builtin_amdgcn_exp2f(sm[k][0][item] - m);
                        L += f * sm[k][1][item];
                        acc += f * so[k][item];
                    }
                }
                M = m;
            }
            __syncthreads();  // before the next pass writes them again
        }
        if (sg != 0 || !in_row) continue;
        if (M != -INFINITY) {
            L += sink_term(a.sinks, g * a.group + rr % a.group, M);
            acc *= 1.f / L;
        }
        const int j = rr / a.group, gh = rr - j * a.group;
        const int64_t hrow = (int64_t)(rq.q0 + j) * a.hq + g * a.group + gh;
        *reinterpret_cast<uint2*>(out + hrow * D + d0) =
            make_uint2(pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]));
    }
}

// ------------------------------------------------------------------ combine
//
// One wavefront per (query row, q-head): merge of the split partials, O = sum_s
// 2^(m_s - M) o_s / sum_s 2^(m_s - M) l_s with M the largest m_s.  Also writes the
// zero output of rows whose request has no key at all.
// A split leaves its sums and the maximum they are relative to.  With normalised
// outputs and log-sum-exps in their place every split's weight had the rounding of
// a logarithm of the size of the scores (error against 64 bits of small calls,
// which are cut into many splits, 1.87e-7 -> 1.66e-7, of 16 requests of 1k to 8k
// tokens 3.56e-7 -> 2.85e-7; the same time).
// The maxima and sums of up to 64 splits are read together, one per lane, and the
// partials eight at a time, all of a round's loads before their use: with one
// load per split behind the test of its maximum the merge of 33 splits was a
// chain of memory latencies (2560 rows: 19.9 us).
template <int D>
__global__ __launch_bounds__(kAttnThreads) void attn_combine(AttnArgs a, int total_q) {
    constexpr int DPL = D / kWave;
    constexpr int kRound = 8;
    const int64_t item = (int64_t)blockIdx.x * kAttnWaves + threadIdx.x / kWave;
    if (item >= (int64_t)total_q * a.hq) return;
    const int lane = threadIdx.x & (kWave - 1);
    const int row = (int)(item / a.hq);
    // request owning `row`: the largest i with q_start[i] <= row
    int lo = 0, hi = a.num_seqs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.q_start[mid] <= row) lo = mid; else hi = mid - 1;
    }
    const SeqGeom sg = seq_geom(a, lo);
    float* outp = static_cast<float*>(a.out) + item * D + lane * DPL;
    const int h = (int)(item - (int64_t)row * a.hq);
    // rows past the launch's reach (a request with more than max_q_len rows) are
    // not computed: quiet NaN instead of stale memory
    if ((row - sg.q0) * a.group + h % a.group >= a.row_groups * a.rows_per_group) {
#pragma unroll
        for (int e = 0; e < DPL; ++e) outp[e] = __builtin_nanf("");
        return;
    }
    if (sg.nsplit == 1) return;
    float acc[DPL];
#pragma unroll
    for (int e = 0; e < DPL; ++e) acc[e] = 0.f;
    float M = -INFINITY, L = 0.f;
    for (int base = 0; base < sg.nsplit; base += kWave) {
        const int64_t pi0 = item * a.max_splits + base;
        const int ns = min(kWave, sg.nsplit - base);
        f32x2u_t ml = {-INFINITY, 0.f};
        if (lane < ns) ml = *reinterpret_cast<const f32x2u_t*>(a.part_ml + 2 * (pi0 + lane));
        const float mnew = fmaxf(M, wave_max_xor(ml.x, kWave));
        if (mnew == -INFINITY) continue;
        // rescale what earlier splits summed (nothing yet: M = -inf gives 0)
        const float alpha = exp2f(M - mnew);
        const float f = exp2f(ml.x - mnew);
        L = L * alpha + wave_sum_xor(f * ml.y, kWave);
#pragma unroll
        for (int e = 0; e < DPL; ++e) acc[e] *= alpha;
        M = mnew;
        const float* po = a.part_o + pi0 * D + lane * DPL;
        for (int s0 = 0; s0 < ns; s0 += kRound) {
            float v[kRound][DPL];
#pragma unroll
            for (int k = 0; k < kRound; ++k)
#pragma unroll
                for (int e = 0; e < DPL; ++e) v[k][e] = po[(int64_t)min(s0 + k, ns - 1) * D + e];
#pragma unroll
            for (int k = 0; k < kRound; ++k) {
                // splits past the last have f = 0 (m -inf); at 64 the lane wraps
                const float fk = s0 + k < ns ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), s0 + k)) : 0.f;
#pragma unroll
                for (int e = 0; e < DPL; ++e) acc[e] = fmaf(fk, v[k][e], acc[e]);
            }
        }
    }
    if (M != -INFINITY) L += sink_term(a.sinks, h, M);
#pragma unroll
    for (int e = 0; e < DPL; ++e) outp[e] = L > 0.f ? acc[e] / L : 0.f;
}

// ------------------------------------------------------------------ KV append
//
// The verify step's new tokens (row j of request i sits at position
// p = S_i - n_i + j) get their K and V written into slot p % 16 of block
// block_tables[i][p / 16]: K x-packed ([D/x][16][x] per block and head), V
// transposed ([D][16]).  One workgroup per (request, KV head) writes all of
// the request's new tokens of that head, so the tokens that share a 32-byte
// V sector (consecutive slots of one dimension) are written by one compute
// unit and leave its L2 as one sector.  Tokens with a negative position or a
// block id outside [0, num_blocks) are skipped.
//
// The call is a chain of memory latencies (its bytes take under a microsecond),
// so each is paid once: kAppendTokens tokens at a time, the rows are read whole
// into LDS (16 bytes per thread, rows contiguous) beside the block ids, and
// leave it transposed, thread items ordered so that consecutive threads write
// consecutive slots: K in 16-byte chunks, V element by element.  Read by
// element in the order of the writes, with the block id looked up for each, the
// loop over dimensions paid the latency over and over (64 requests of 1 to 17
// tokens, 8 heads of 128: 9.7 -> 6.5 us).
constexpr int kAppendThreads = 256;
constexpr int kAppendTokens = 32;

template <typename T, int D>
__global__ __launch_bounds__(kAppendThreads) void attn_kv_append(
    int num_seqs, int hkv, int max_blocks, int num_blocks, const T* __restrict__ k_new,
    const T* __restrict__ v_new, const int32_t* __restrict__ block_tables,
    const int32_t* __restrict__ seq_lens, const int32_t* __restrict__ q_start, T* __restrict__ kc,
    T* __restrict__ vc) {
    constexpr int X = Storage<T>::kPer16B;
    constexpr int NC = D / X;  // 16-byte chunks per key
    // rows of NC chunks, one more per row so that the reads down a column of
    // consecutive tokens spread over the banks
    __shared__ uint4 ks[kAppendTokens][NC + 1], vs[kAppendTokens][NC + 1];
    __shared__ int32_t blk[kAppendTokens];
    const int i = blockIdx.x, g = blockIdx.y, tid = threadIdx.x;
    const int q0 = q_start[i];
    const int n = q_start[i + 1] - q0;
    if (n <= 0) return;
    const int64_t p0 = (int64_t)seq_lens[i] - n;  // position of the request's row 0
    const int32_t* bt = block_tables + (int64_t)i * max_blocks;
    // rows that a caller aligned to their elements only are read by element
    const bool wide = (((uintptr_t)k_new | (uintptr_t)v_new) & 15) == 0;
    for (int j0 = 0; j0 < n; j0 += kAppendTokens) {
        const int m = min(kAppendTokens, n - j0);
        if (j0 > 0) __syncthreads();
        const T* kr = k_new + ((int64_t)(q0 + j0) * hkv + g) * D;
        const T* vr = v_new + ((int64_t)(q0 + j0) * hkv + g) * D;
        const int64_t stride = (int64_t)hkv * D;
        if (wide) {
#pragma unroll
            for (int u = 0; u < kAppendTokens * NC / kAppendThreads; ++u) {
                const int it = u * kAppendThreads + tid, j = it / NC, c = it % NC;
                if (j < m) {
                    ks[j][c] = ld16(kr + j * stride + c * X);
                    vs[j][c] = ld16(vr + j * stride + c * X);
                }
            }
        } else {
            for (int it = tid; it < m * D; it += kAppendThreads) {
                const int j = it / D, d = it % D;
                reinterpret_cast<T*>(ks[j])[d] = kr[j * stride + d];
                reinterpret_cast<T*>(vs[j])[d] = vr[j * stride + d];
            }
        }
        if (tid < m) {
            const int64_t p = p0 + j0 + tid;
            int b = -1;
            if (p >= 0 && p / kBlockTokens < max_blocks) b = bt[p / kBlockTokens];
            blk[tid] = b >= 0 && b < num_blocks ? b : -1;
        }
        __syncthreads();
        // tokens fastest, over the next power of two of them
        const int sh = m > 1 ? 32 - __clz(m - 1) : 0;
        const int j = tid & ((1 << sh) - 1), step = kAppendThreads >> sh;
        const int b = j < m ? blk[j] : -1;
        if (b >= 0) {
            const int t = (int)((p0 + j0 + j) % kBlockTokens);
            const int64_t tile = ((int64_t)b * hkv + g) * D * kBlockTokens;
            for (int c = tid >> sh; c < NC; c += step)
                *reinterpret_cast<uint4*>(kc + tile + (c * kBlockTokens + t) * X) = ks[j][c];
            for (int d = tid >> sh; d < D; d += step)
                vc[tile + d * kBlockTokens + t] = reinterpret_cast<const T*>(vs[j])[d];
        }
    }
}

// ------------------------------------------------------------------ host side

struct AttnPlan {
    bool mfma;        // bf16 storage: persistent kernel; fp32 storage: split-K kernel
    // fp32 path
    int split_blocks;
    int max_splits;
    int row_groups;
    int tiles;        // 16-row tiles per work item
    size_t part_o_bytes;
    size_t part_ml_bytes;
    // bf16 path: one persistent launch per row class
    struct Class {
        int nw, tpw;          // wavefronts per workgroup, 16-row tiles per wavefront
        int rg_max;           // row groups per (request, KV head)
        int nwg;              // persistent workgroups
        int spb;              // fixed units per workgroup (0: equal shares)
        bool whole;           // one workgroup per pair
        bool slot_f32;        // the partial outputs are fp32
        int rows_lo, rows_hi; // requests with Hq/Hkv * n_i in [rows_lo, rows_hi]
        int64_t slots;        // partial slots
        size_t off;           // workspace offset of the class's arrays
        size_t unit_bytes, slot_o_bytes, slot_lse_bytes;
        size_t cover_bytes;   // what the class needs at most with fewer requests
    };
    int nclass;
    Class cls[2];
    size_t total_bytes;       // workspace of the call
    // workspace that the size query returns: enough for any call of fewer
    // requests too.  A caller keeps one workspace for its largest batch, and a
    // smaller one can need more of it: its pairs are cut where those of the
    // largest fill the chip whole, and into more ranges.
    size_t cover_bytes;
};

// Batches whose requests carry up to this many query rows per KV head (three
// 16-row tiles) and more than that run in two launches, each with its own
// kernel shape (see make_plan).
constexpr int kShortClassRows = 48;

// A launch whose workgroups would each own more than this many units (each
// unit a 16-token block of 8 KiB at head dim 128, so about 3 ms of streaming)
// launches up to eight times the resident workgroups: the hardware hands the
// next workgroup to whichever compute unit frees a slot first, so faster
// compute units take more of the work (long-context batch: 10.06 -> 9.10 ms at
// eight times; at the short Qwen and DSK calls the extra start-ups cost more
// than the balance gains).
constexpr int64_t kOversubUnits = 4096;

// Ranges that a plan of few pairs cuts a pair of the longest length into.  More
// workgroups shorten the walk (0.28 us per block and workgroup on an idle chip),
// but each adds a slot per pair that the merge reads, 32 of them in a round of
// about 1.1 us where four thread groups share a row.  The sum is least at
// sqrt(8.2 blocks) ranges: 28 of 95 blocks, 91 of 1001, 259 of 8188.  Measured
// on one request (us for 24 / 32 / 48 / 64 / 96 / 128 / 192 / 256 ranges; eight
// KV heads: 251 blocks 16.8 / 16.6 / 17.3 / 16.7 / 17.8; 1001 blocks 29.1 / 27.3 /
// 26.4 / 26.8 / 25.4 / 27.3 / 31.8 / 36.3; one KV head, 8188 blocks 210 / 161 /
// 114 / 90 / 67 / 57 / 47 / 43).  Beyond about two thirds of the resident
// workgroups in the launch more of them only lengthen the merge (32 pairs of 1001
// blocks: 52 us with 768, 54 with 1024, 60 with 2048).  Multiples of 30, so that
// a pair with a range boundary off its ends still has whole rounds of slots; at
// least kMinRanges (95 blocks: 13.7 us with 24 ranges, 14.4 with 16), and no range
// planned below two blocks.  These are the plan's figures, for pairs as long as
// the longest may be: where lengths differ, a long pair gets more than its share
// of the ranges, and where they all are shorter, ranges of one block occur.
constexpr int kMinRanges = 24;

int64_t ranges_per_pair(int64_t nb_max, int64_t pairs, int64_t resident) {
    const int64_t best = std::min((int64_t)std::sqrt(8.2 * (double)nb_max), 2 * resident / (3 * pairs));
    return best < 30 ? kMinRanges : best / 30 * 30;
}

// Whether a launch gives every pair to one workgroup: no schedule scan, no
// partial slots and no merge launch, at the price of a walk as long as the
// longest pair.  Up to 16 blocks whole pairs are always faster (8 KV heads of one
// request, 16 blocks: 10.2 against 10.7 us, 32 blocks 14.7 against 9.5 us).
// Beyond that they are where the pairs fill the compute units and their lengths
// are alike: 256 pairs of 32 blocks 20.2 against 28.8 us, 512 of 88 blocks 64
// against 86.  But the plan does not see the lengths, and the longest pair may be
// long alone; the lines lie where that costs what the cut walk does.  One request
// at the longest length among requests of two or three blocks, whole against cut:
//   one wavefront: 17 blocks 12 against 13 us, 26 to 33 16.6 against 15.7, 40
//     18 against 14, 64 25 against 17;
//   several of one tile: 64 blocks 24 against 33 us, 88 blocks 25 to 31 against
//     35 to 43;
//   several of more tiles: 64 blocks 42 against 62 us, 88 blocks 45 to 55 against
//     41 to 48.
// With fewer pairs the line comes down to the 16 blocks (30 pairs of 21 blocks and
// up to eight tiles 38.6 whole against 36.2 us).  pairs counts those that can
// have rows: a launch of long rows is not filled by the requests of the other one.
bool whole_pairs(int64_t nb_max, int64_t pairs, int64_t cus, int nw, int tpw) {
    if (nb_max <= 16) return true;
    const int64_t most = nw == 1 ? 28 : tpw == 1 ? 95 : 72;
    return 2 * pairs >= cus && nb_max <= std::min(most, 16 + 48 * pairs / cus);
}

// LDS stages (blocks) of a workgroup's ring.  A step computes two of them while
// the others load.  Five (40 KiB at D = 128, 20 KiB at D = 64) let four (eight)
// workgroups share a compute unit's 160 KiB of LDS, which is why the schedule
// scan borrows the last stage instead of LDS of its own.  The four-wavefront
// two-tile shape fits three workgroups by its registers and takes six.  More
// workgroups per compute unit beat deeper rings (six stages and three
// workgroups: 985 against 860 us on 4.6 GB at D = 64), and with four stages a
// step finds nothing in flight behind its own blocks (284 against 239 us on
// 1.2 GB at D = 128).
constexpr int ring_stages(int d, int nw, int tpw) { return d == 128 && nw == 4 && tpw == 2 ? 6 : 5; }

// The kernel shapes a plan may choose: head dim, wavefronts per workgroup,
// 16-row tiles per wavefront.  with_shape calls f(Shape<...>{}) for the
// matching entry and returns false if there is none.
template <int D_, int NW_, int TPW_>
struct Shape {
    static constexpr int D = D_, NW = NW_, TPW = TPW_, NS = ring_stages(D_, NW_, TPW_);
};

template <typename F>
bool with_shape(int d, int nw, int tpw, F&& f) {
#define AVERIFY_SHAPE(D_, NW_, TPW_)                       \
    if (d == D_ && nw == NW_ && tpw == TPW_) {             \
        f(Shape<D_, NW_, TPW_>{});                         \
        return true;                                       \
    }
    AVERIFY_SHAPE(128, 1, 1)
    AVERIFY_SHAPE(128, 1, 3)
    AVERIFY_SHAPE(128, 2, 1)
    AVERIFY_SHAPE(128, 2, 2)
    AVERIFY_SHAPE(128, 4, 2)
    AVERIFY_SHAPE(64, 1, 1)
    AVERIFY_SHAPE(64, 1, 5)
    AVERIFY_SHAPE(64, 2, 1)
    AVERIFY_SHAPE(64, 4, 1)
    AVERIFY_SHAPE(64, 4, 2)
    AVERIFY_SHAPE(64, 4, 3)
    AVERIFY_SHAPE(64, 4, 4)
#undef AVERIFY_SHAPE
    return false;
}

template <typename S, bool APPEND = false, typename Slot = uint16_t>
constexpr auto persist_kernel() {
    return attn_persist<S::D, S::NW, S::TPW, S::NS, APPEND, Slot>;
}

int validate(const verify_attn_params* p, int32_t total_q, int32_t max_q_len,
             int32_t max_seq_len) {
    if (!p) return VERIFY_EINVAL;
    if (p->dtype != VERIFY_F32 && p->dtype != VERIFY_BF16) return VERIFY_EUNSUPPORTED;
    if (p->head_dim != 64 && p->head_dim != 128) return VERIFY_EUNSUPPORTED;
    if (p->block_size != kBlockTokens) return VERIFY_EUNSUPPORTED;
    if (p->num_seqs < 0 || p->num_q_heads <= 0 || p->num_kv_heads <= 0) return VERIFY_EINVAL;
    if (p->num_q_heads % p->num_kv_heads != 0) return VERIFY_EINVAL;
    if (p->max_blocks_per_seq <= 0 || p->num_blocks < 0 || p->sliding_window < 0) return VERIFY_EINVAL;
    if (p->kv_split_blocks < 0 || !(p->scale >= 0.f) || p->scale > 3.0e38f) return VERIFY_EINVAL;
    if (total_q < 0 || max_q_len < 0 || max_seq_len < 0) return VERIFY_EINVAL;
    if (p->num_seqs > 65535) return VERIFY_EUNSUPPORTED;
    return VERIFY_OK;
}

// Compute units of the current device and resident workgroups per compute
// unit of a kernel (cached per device; fallbacks when no device is visible).
int device_cus() {
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { (void)hipGetLastError(); return 256; }
    int v = cache[dev].load(std::memory_order_relaxed);
    if (v > 0) return v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) {
        (void)hipGetLastError();
        v = 256;
    }
    cache[dev].store(v, std::memory_order_relaxed);
    return v;
}

template <typename S, bool APPEND = false>
int resident_wgs() {
    static std::atomic<int> cache[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) { (void)hipGetLastError(); return 2; }
    int v = cache[dev].load(std::memory_order_relaxed);
    if (v > 0) return v;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, persist_kernel<S, APPEND>(), S::NW * kWave, 0) !=
            hipSuccess ||
        v <= 0) {
        (void)hipGetLastError();
        v = 1;
    }
    cache[dev].store(v, std::memory_order_relaxed);
    return v;
}

// Kernel shape (wavefronts per workgroup, tiles per wavefront) for row groups
// of up to `tiles` 16-row tiles.  A single tile goes to single-wavefront
// workgroups: every wavefront is an independent worker with its own LDS ring
// and no barrier.  More rows use NW wavefronts sharing one ring (NW divides
// the 16-byte chunks of a block, 512 at D = 128 and 256 at D = 64, so every
// thread loads alike).  At D = 128 a wavefront takes two tiles once there are
// three or more: fewer wavefronts per block mean fewer barriers and more
// workgroups per compute unit, which is what hides the per-block latency of
// the online softmax.  Rows beyond the shape's reach are split into row
// groups, each walking the request's KV again.
void pick_shape(int head_dim, int64_t tiles, int64_t nb_max, int& nw, int& tpw) {
    if (tiles <= 1) {
        nw = 1;
        tpw = 1;
    } else if (head_dim == 128) {
        nw = tiles <= 4 ? 2 : 4;
        tpw = tiles == 2 ? 1 : 2;
        if (tiles == 3 && nb_max >= 64) { nw = 1; tpw = 3; }
    } else {
        nw = tiles <= 2 ? 2 : 4;
        tpw = (int)std::min<int64_t>(4, (tiles + nw - 1) / nw);
        if (tiles == 5 && nb_max >= 64) { nw = 1; tpw = 5; }
    }
}

// The persistent launch of one row class: requests with rows_lo <= Hq/Hkv *
// n_i <= rows_hi, of which no request has more than `rows` rows.
int plan_class(const verify_attn_params* p, int32_t total_q, int64_t rows, int64_t nb_max, int rows_lo,
               int rows_hi, bool append, AttnPlan::Class& c) {
    c = AttnPlan::Class{};
    pick_shape(p->head_dim, (rows + 15) / 16, nb_max, c.nw, c.tpw);
    c.rows_lo = rows_lo;
    c.rows_hi = rows_hi;
    const int64_t per = (int64_t)c.nw * c.tpw * 16;
    c.rg_max = (int)((rows + per - 1) / per);
    const int64_t pairs = (int64_t)std::max(1, p->num_seqs) * p->num_kv_heads * c.rg_max;
    // of which so many at most have rows in the class
    const int64_t active = rows_lo > 0 ? (int64_t)total_q * (p->num_q_heads / p->num_kv_heads) / rows_lo *
                                             p->num_kv_heads * c.rg_max
                                       : pairs;
    const int64_t units_max = pairs * nb_max;
    if (units_max >= (int64_t)1 << 31) return VERIFY_EUNSUPPORTED;
    c.spb = p->kv_split_blocks;
    int64_t all = 0;  // resident workgroups
    if (c.spb > 0) {
        c.nwg = (int)std::min<int64_t>((units_max + c.spb - 1) / c.spb, (int64_t)1 << 30);
    } else {
        int res = 0;
        // the fused-append kernel holds more registers, and may fit fewer
        // workgroups per compute unit
        if (!with_shape(p->head_dim, c.nw, c.tpw, [&](auto sh) {
                res = append ? resident_wgs<decltype(sh), true>() : resident_wgs<decltype(sh)>();
            }))
            return VERIFY_EUNSUPPORTED;
        all = (int64_t)device_cus() * res;
        const int64_t ranges = ranges_per_pair(nb_max, pairs, all);
        const int64_t apart = std::max<int64_t>(2, (nb_max + ranges - 1) / ranges);
        const int64_t resident = std::min(all, (units_max + apart - 1) / apart);
        c.slot_f32 = resident < all;
        const int64_t mult = std::min<int64_t>(8, std::max<int64_t>(1, units_max / resident / kOversubUnits));
        c.nwg = (int)(resident * mult);
    }
    c.slots = pairs + c.nwg;
    // slots with fewer requests: no more pairs and workgroups than these (nwg
    // before it is capped by the units), fp32 only in launches of fewer than `all`
    int64_t most = c.slots, most_f32 = 0;
    if (c.spb == 0) {
        most = pairs + std::min(8 * all, std::max(all, units_max / kOversubUnits));
        most_f32 = std::min(pairs, all) + all;
    }
    if (c.spb == 0 && whole_pairs(nb_max, std::min(pairs, active), device_cus(), c.nw, c.tpw)) {
        c.whole = true;
        c.nwg = (int)pairs;
        c.slots = 0;
        c.slot_f32 = false;
    }
    c.unit_bytes = align_up(sizeof(int32_t) * ((size_t)std::max(1, p->num_seqs) + 1), 256);
    c.slot_o_bytes = align_up((size_t)c.slots * per * p->head_dim * (c.slot_f32 ? sizeof(float) : sizeof(uint16_t)), 256);
    c.slot_lse_bytes = align_up((size_t)c.slots * per * sizeof(float), 256);
    const size_t values = (size_t)per * p->head_dim;
    c.cover_bytes = c.unit_bytes + align_up(std::max(most * values * sizeof(uint16_t), most_f32 * values * sizeof(float)), 256) +
                    align_up((size_t)std::max(most, most_f32) * per * sizeof(float), 256);
    // (a launch of few, very long pairs is oversubscribed past most_f32)
    c.cover_bytes = std::max(c.cover_bytes, c.unit_bytes + c.slot_o_bytes + c.slot_lse_bytes);
    return VERIFY_OK;
}

// fp32 storage: a split is at most kF32SplitBlocks blocks (a partial row of D
// floats per split is written and read again: 16 requests of 1k to 8k tokens take
// 163 / 152 / 155 / 148 / 175 us at 16 / 24 / 32 / 48 / 64, and long splits leave
// the last workgroups alone), shorter when the batch has fewer than kF32Items of
// them (a workgroup per compute unit), down to a block per wavefront: one request
// of 94 blocks 28 us at 32, under the call's host time from 16 down; two requests
// of 3750 blocks on one KV head 63 / 45 / 38 / 39 / 56 us at 8 / 16 / 24 / 32 / 64.
// From 262144 blocks on the items are held to about kF32MostItems.
constexpr int kF32Items = 256;
constexpr int kF32MostItems = 8192;
constexpr int kF32SplitBlocks = 32;

int make_plan(const verify_attn_params* p, int32_t total_q, int32_t max_q_len,
              int32_t max_seq_len, AttnPlan* out, bool append = false) {
    AttnPlan pl{};
    const int G = p->num_q_heads / p->num_kv_heads;
    int64_t nb_max = ((int64_t)max_seq_len + kBlockTokens - 1) / kBlockTokens;
    if (p->sliding_window > 0) {
        const int64_t span = (int64_t)p->sliding_window + max_q_len - 1;
        nb_max = std::min<int64_t>(nb_max, (span + kBlockTokens - 1) / kBlockTokens + 1);
    }
    nb_max = std::max<int64_t>(nb_max, 1);
    const int64_t rows = (int64_t)G * std::max(1, max_q_len);
    pl.mfma = p->dtype == VERIFY_BF16;
    if (pl.mfma) {
        // One launch sized by the largest request.  At head dim 128, when that
        // takes the four-wavefront shape (five tiles or more), the requests
        // of up to three tiles get a launch of their own with the shape of
        // three tiles: the four-wavefront shape streams 5.4 TB/s on pairs of
        // one tile but 4.2 TB/s on pairs of eight, and 5.9-6.0 TB/s on pairs
        // of three in the three-tile shape (long contexts), so mixing draft
        // lengths in one launch runs every pair at about the slow rate.
        int rc;
        if (p->head_dim == 128 && (rows + 15) / 16 >= 5) {
            pl.nclass = 2;
            rc = plan_class(p, total_q, kShortClassRows, nb_max, 0, kShortClassRows, append, pl.cls[0]);
            if (rc == VERIFY_OK)
                rc = plan_class(p, total_q, rows, nb_max, kShortClassRows + 1, INT32_MAX, append, pl.cls[1]);
        } else {
            pl.nclass = 1;
            rc = plan_class(p, total_q, rows, nb_max, 0, INT32_MAX, append, pl.cls[0]);
        }
        if (rc != VERIFY_OK) return rc;
        size_t off = 0;
        for (int k = 0; k < pl.nclass; ++k) {
            AttnPlan::Class& c = pl.cls[k];
            c.off = off;
            off += c.unit_bytes + c.slot_o_bytes + c.slot_lse_bytes;
            pl.cover_bytes += c.cover_bytes;
        }
        pl.total_bytes = off;
    } else {
        // as few row groups as hold the tiles, the tiles spread evenly over them
        const int64_t tiles = (rows + 15) / 16, most = f32_max_tiles(p->head_dim);
        pl.row_groups = (int)std::min<int64_t>((tiles + most - 1) / most, 1 << 24);
        pl.tiles = (int)((tiles + pl.row_groups - 1) / pl.row_groups);
        int sb = p->kv_split_blocks;
        if (sb == 0) {
            const int64_t total = (int64_t)std::max(1, p->num_seqs) * p->num_kv_heads * pl.row_groups * nb_max;
            int64_t want = ((total + kF32Items - 1) / kF32Items + 3) / 4 * 4;
            want = std::min<int64_t>(want, std::max<int64_t>(kF32SplitBlocks, (total / kF32MostItems + 3) / 4 * 4));
            sb = (int)std::min<int64_t>(want, nb_max);
        }
        pl.split_blocks = std::max(1, sb);
        pl.max_splits = (int)((nb_max + pl.split_blocks - 1) / pl.split_blocks);
        // the call's limit since its grid had a 16-bit dimension of row groups of
        // eight rows; the walk's (pairs x splits, requests) needs fewer than 2^24
        // pairs, which it implies
        if ((int64_t)p->num_kv_heads * ((rows + 7) / 8) > 65535) return VERIFY_EUNSUPPORTED;
        if (pl.max_splits > 1) {
            const size_t items = (size_t)total_q * p->num_q_heads * pl.max_splits;
            pl.part_o_bytes = align_up(items * p->head_dim * sizeof(float), 256);
            pl.part_ml_bytes = align_up(items * 2 * sizeof(float), 256);
        }
        pl.total_bytes = pl.part_o_bytes + pl.part_ml_bytes;
        pl.cover_bytes = pl.total_bytes;
        if (p->kv_split_blocks == 0 && nb_max > 4) {
            // (rows, splits) of b requests, over all b: rows t <= total_q and t <= b
            // max_q_len.  A split has at least total / kF32Items blocks (total is
            // proportional to b), or kF32SplitBlocks and total / kF32MostItems of
            // which rounding down takes less than one in 33, so t * splits is at
            // most t + max_q_len * items / (KV heads * row groups).
            const int64_t t = total_q, walks = (int64_t)p->num_kv_heads * pl.row_groups;
            auto most = [&](int64_t items, int64_t blocks) {
                return std::min(t * ((nb_max + blocks - 1) / blocks),
                                t + ((int64_t)std::max(1, max_q_len) * items + walks - 1) / walks);
            };
            const size_t rows_splits = (size_t)std::max(most(kF32Items, 4), most(kF32MostItems * 33 / 32, kF32SplitBlocks));
            const size_t part = rows_splits * p->num_q_heads;
            pl.cover_bytes = std::max(pl.total_bytes, align_up(part * p->head_dim * sizeof(float), 256) +
                                                          align_up(part * 2 * sizeof(float), 256));
        }
    }
    *out = pl;
    return VERIFY_OK;
}

// Schedule pass, then the persistent kernel of the plan's shape, then the
// merge of partial slots.  Returns false if the plan names no known shape.
bool launch_persist(const PArgs& a, const MPtrs& m, const AttnPlan::Class& pl, int head_dim,
                    int max_rows, hipStream_t stream) {
    return with_shape(head_dim, pl.nw, pl.tpw, [&](auto sh) {
        using S = decltype(sh);
        if (!a.inline_sched && !a.whole)
            hipLaunchKernelGGL((attn_schedule<S::D>), dim3(1), dim3(1024), 0, stream, a, m.q_start,
                               m.seq_lens, m.unit_start, m.out);
        auto walk = [&](auto append, auto slot) {
            using Slot = decltype(slot);
            hipLaunchKernelGGL((persist_kernel<S, decltype(append)::value, Slot>()), dim3(a.nwg),
                               dim3(S::NW * kWave), 0, stream, a, m.q, m.kc, m.vc, m.block_tables, m.seq_lens,
                               m.q_start, m.unit_start, m.out, static_cast<Slot*>(m.slot_o), m.slot_lse, m.k_new,
                               m.v_new);
        };
        if (m.k_new) pl.slot_f32 ? walk(std::true_type{}, float{}) : walk(std::true_type{}, uint16_t{});
        else pl.slot_f32 ? walk(std::false_type{}, float{}) : walk(std::false_type{}, uint16_t{});
        if (a.whole) return;
        const int64_t pairs = (int64_t)a.num_seqs * a.hkv * a.rg_max;
        // rows of a row group: at most rows_per_group, at most G * max_q_len
        const int group_rows = std::max(1, std::min(a.rows_per_group, max_rows));
        auto combine = [&](auto sg, auto slot) {
            using Slot = decltype(slot);
            constexpr int SG = decltype(sg)::value, RPB = kCombineThreads / (S::D / 4) / SG;
            const unsigned chunks = (unsigned)((group_rows + RPB - 1) / RPB);
            hipLaunchKernelGGL((attn_combine_slots<S::D, SG, Slot>), dim3((unsigned)pairs, chunks),
                               dim3(kCombineThreads), 0, stream, a, m.seq_lens, m.q_start,
                               m.unit_start, static_cast<const Slot*>(m.slot_o), m.slot_lse, m.out);
        };
        if (pairs <= 0) return;
        // more than one and a half rounds of slots per planned pair (the average; a
        // long pair among short ones has more): four thread groups share a row, if the four times larger grid is resident at once (88 pairs of 52
        // rows in 14 slots 26.5 -> 23.0 us, but 41 pairs of 240 rows in 12 slots 30.2
        // -> 34.7, 30 pairs of 88 rows in 10 slots 36.2 -> 38.6)
        const int64_t wgs4 = pairs * ((group_rows * S::D + kCombineThreads - 1) / kCombineThreads);
        const std::integral_constant<int, 1> alone;
        const std::integral_constant<int, 4> shared;
        const bool share = 2 * (int64_t)a.nwg > 3 * kCombineSlots * pairs && wgs4 <= 8 * (int64_t)device_cus();
        if (pl.slot_f32) share ? combine(shared, float{}) : combine(alone, float{});
        else share ? combine(shared, uint16_t{}) : combine(alone, uint16_t{});
    });
}

template <int D>
void launch_f32(AttnArgs a, const AttnPlan& pl, int total_q, hipStream_t stream) {
    // a grid dimension holds fewer than 2^32 threads, 2^24 workgroups
    const int pairs = a.hkv * pl.row_groups, step = ((1 << 24) - 1) / pairs;
    dim3 grid(1, a.num_seqs);
    auto walk = [&](auto rt) {
        constexpr int RT = decltype(rt)::value;
        if (a.k_new) hipLaunchKernelGGL((attn_f32<D, RT, true>), grid, dim3(kAttnThreads), 0, stream, a);
        else hipLaunchKernelGGL((attn_f32<D, RT, false>), grid, dim3(kAttnThreads), 0, stream, a);
    };
    for (a.split0 = 0; a.split0 < pl.max_splits; a.split0 += step) {
        grid.x = (unsigned)std::min(step, pl.max_splits - a.split0) * pairs;
        if (pl.tiles == 1) walk(std::integral_constant<int, 1>{});
        else if (pl.tiles == 2) walk(std::integral_constant<int, 2>{});
        else if (pl.tiles == 3) walk(std::integral_constant<int, 3>{});
        else walk(std::integral_constant<int, f32_max_tiles(D)>{});
    }
    const int64_t items = (int64_t)total_q * a.hq;
    if (items > 0) {
        dim3 cgrid((unsigned)((items + kAttnWaves - 1) / kAttnWaves));
        hipLaunchKernelGGL((attn_combine<D>), cgrid, dim3(kAttnThreads), 0, stream, a, total_q);
    }
}

}  // namespace
}  // namespace averify

using namespace averify;

extern "C" int verify_attention_workspace_size(const verify_attn_params* params, int32_t total_q,
                                               int32_t max_q_len, int32_t max_seq_len,
                                               size_t* bytes) {
    if (!bytes) return VERIFY_EINVAL;
    int rc = validate(params, total_q, max_q_len, max_seq_len);
    if (rc != VERIFY_OK) return rc;
    // enough for verify_attention and verify_attention_append alike
    AttnPlan pl, pla;
    rc = make_plan(params, total_q, max_q_len, max_seq_len, &pl);
    if (rc == VERIFY_OK) rc = make_plan(params, total_q, max_q_len, max_seq_len, &pla, true);
    if (rc != VERIFY_OK) return rc;
    *bytes = std::max(pl.cover_bytes, pla.cover_bytes);
    return VERIFY_OK;
}

namespace {

// verify_attention, and with k_new / v_new non-null verify_attention_append
int attention_call(const verify_attn_params* params, int32_t total_q, int32_t max_q_len,
                   int32_t max_seq_len, const void* q, const void* k_cache, const void* v_cache,
                   const int32_t* block_tables, const int32_t* seq_lens, const int32_t* q_start,
                   const float* sinks, void* out, void* workspace, size_t workspace_bytes,
                   const void* k_new, const void* v_new, hipStream_t stream) {
    int rc = validate(params, total_q, max_q_len, max_seq_len);
    if (rc != VERIFY_OK) return rc;
    const verify_attn_params& p = *params;
    if (p.num_seqs > 0 && (!seq_lens || !q_start || !block_tables)) return VERIFY_EINVAL;
    if (total_q > 0 && (!q || !k_cache || !v_cache || !out)) return VERIFY_EINVAL;
    // a query row sits at a position of its own request, so its cache holds
    // at least one block
    if (total_q > 0 && p.num_blocks < 1) return VERIFY_EINVAL;
    AttnPlan pl;
    rc = make_plan(params, total_q, max_q_len, max_seq_len, &pl, k_new != nullptr);
    if (rc != VERIFY_OK) return rc;
    if (workspace_bytes < pl.total_bytes || (pl.total_bytes > 0 && !workspace)) return VERIFY_EWORKSPACE;
    if (p.num_seqs == 0 || total_q == 0) return VERIFY_OK;
    const float scale = p.scale > 0.f ? p.scale : 1.0f / sqrtf((float)p.head_dim);

    if (pl.mfma) {
        MPtrs m{};
        m.q = static_cast<const uint16_t*>(q);
        m.kc = static_cast<const uint8_t*>(k_cache);
        m.vc = static_cast<const uint8_t*>(v_cache);
        m.block_tables = block_tables;
        m.seq_lens = seq_lens;
        m.q_start = q_start;
        m.out = static_cast<uint16_t*>(out);
        m.k_new = static_cast<const uint16_t*>(k_new);
        m.v_new = static_cast<const uint16_t*>(v_new);
        PArgs a{};
        a.num_seqs = p.num_seqs;
        a.hq = p.num_q_heads;
        a.hkv = p.num_kv_heads;
        a.group = p.num_q_heads / p.num_kv_heads;
        a.max_blocks = p.max_blocks_per_seq;
        a.num_blocks = p.num_blocks;
        a.window = p.sliding_window;
        a.max_seq_len = max_seq_len;
        a.scale_log2 = scale * kLog2e;
        a.inv_scale_log2 = a.scale_log2 > 0.f ? 1.f / a.scale_log2 : 0.f;
        a.inline_sched = p.num_seqs <= kInlineSchedSeqs;
        a.sinks = sinks;
        const int64_t max_rows = (int64_t)a.group * std::max(1, max_q_len);
        // one launch per row class, one after another on the stream; each
        // writes only its own requests' outputs
        for (int k = 0; k < pl.nclass; ++k) {
            const AttnPlan::Class& c = pl.cls[k];
            char* ws = static_cast<char*>(workspace) + c.off;
            m.unit_start = reinterpret_cast<int32_t*>(ws);
            m.slot_o = ws + c.unit_bytes;
            m.slot_lse = reinterpret_cast<float*>(ws + c.unit_bytes + c.slot_o_bytes);
            a.rows_per_group = c.nw * c.tpw * 16;
            a.rg_max = c.rg_max;
            a.nwg = c.nwg;
            a.spb = c.spb;
            a.whole = c.whole;
            a.rows_lo = c.rows_lo;
            a.rows_hi = c.rows_hi;
            const int64_t class_rows = std::min<int64_t>(max_rows, c.rows_hi);
            if (!launch_persist(a, m, c, p.head_dim, (int)std::min<int64_t>(class_rows, 1 << 30), stream))
                return VERIFY_EUNSUPPORTED;
        }
        return check_launch();
    }

    AttnArgs a{};
    a.q = q;
    a.kc = k_cache;
    a.vc = v_cache;
    a.block_tables = block_tables;
    a.seq_lens = seq_lens;
    a.q_start = q_start;
    a.out = out;
    a.part_o = pl.part_o_bytes ? static_cast<float*>(workspace) : nullptr;
    a.part_ml = pl.part_o_bytes
                    ? reinterpret_cast<float*>(static_cast<char*>(workspace) + pl.part_o_bytes)
                    : nullptr;
    a.num_seqs = p.num_seqs;
    a.hq = p.num_q_heads;
    a.hkv = p.num_kv_heads;
    a.group = p.num_q_heads / p.num_kv_heads;
    a.max_blocks = p.max_blocks_per_seq;
    a.num_blocks = p.num_blocks;
    a.window = p.sliding_window;
    a.max_seq_len = max_seq_len;
    a.scale_log2 = scale * kLog2e;
    a.split_blocks = pl.split_blocks;
    a.max_splits = pl.max_splits;
    a.row_groups = pl.row_groups;
    a.rows_per_group = pl.tiles * 16;
    a.sinks = sinks;
    a.k_new = k_new;
    a.v_new = v_new;
    if (p.head_dim == 128) launch_f32<128>(a, pl, total_q, stream);
    else launch_f32<64>(a, pl, total_q, stream);
    return check_launch();
}

}  // namespace

extern "C" int verify_attention(const verify_attn_params* params, int32_t total_q,
                                int32_t max_q_len, int32_t max_seq_len, const void* q,
                                const void* k_cache, const void* v_cache,
                                const int32_t* block_tables, const int32_t* seq_lens,
                                const int32_t* q_start, const float* sinks, void* out,
                                void* workspace, size_t workspace_bytes, hipStream_t stream) {
    return attention_call(params, total_q, max_q_len, max_seq_len, q, k_cache, v_cache,
                          block_tables, seq_lens, q_start, sinks, out, workspace, workspace_bytes,
                          nullptr, nullptr, stream);
}

extern "C" int verify_attention_append(const verify_attn_params* params, int32_t total_q,
                                       int32_t max_q_len, int32_t max_seq_len, const void* q,
                                       const void* k_new, const void* v_new, void* k_cache,
                                       void* v_cache, const int32_t* block_tables,
                                       const int32_t* seq_lens, const int32_t* q_start,
                                       const float* sinks, void* out, void* workspace,
                                       size_t workspace_bytes, hipStream_t stream) {
    if (total_q > 0 && (!k_new || !v_new)) return VERIFY_EINVAL;
    return attention_call(params, total_q, max_q_len, max_seq_len, q, k_cache, v_cache,
                          block_tables, seq_lens, q_start, sinks, out, workspace, workspace_bytes,
                          total_q > 0 ? k_new : nullptr, total_q > 0 ? v_new : nullptr, stream);
}

extern "C" int verify_attention_plan(const verify_attn_params* params, int32_t total_q,
                                     int32_t max_q_len, int32_t max_seq_len, int32_t* info) {
    if (!info) return VERIFY_EINVAL;
    int rc = validate(params, total_q, max_q_len, max_seq_len);
    if (rc != VERIFY_OK) return rc;
    AttnPlan pl;
    rc = make_plan(params, total_q, max_q_len, max_seq_len, &pl);
    if (rc != VERIFY_OK) return rc;
    for (int k = 0; k < VERIFY_ATTN_PLAN_INFO; ++k) info[k] = 0;
    if (pl.mfma) {
        info[0] = 1;
        info[5] = pl.nclass;
        for (int k = 0; k < pl.nclass; ++k) {
            const AttnPlan::Class& c = pl.cls[k];
            int32_t* d = k == 0 ? info + 1 : info + 6;
            d[0] = c.nwg;
            d[1] = c.nw * c.tpw * 16;
            d[2] = c.rg_max;
            d[3] = c.whole ? -1 : c.spb;
        }
        info[10] = pl.nclass > 1 ? pl.cls[0].rows_hi : INT32_MAX;
    } else {
        info[0] = 0;
        info[1] = pl.max_splits;
        info[2] = pl.tiles * 16;
        info[3] = pl.row_groups;
        info[4] = pl.split_blocks;
    }
    return VERIFY_OK;
}

extern "C" int verify_kv_append(const verify_attn_params* params, int32_t total_q,
                                const void* k_new, const void* v_new, const int32_t* block_tables,
                                const int32_t* seq_lens, const int32_t* q_start, void* k_cache,
                                void* v_cache, hipStream_t stream) {
    int rc = validate(params, total_q, 0, 0);
    if (rc != VERIFY_OK) return rc;
    const verify_attn_params& p = *params;
    if (total_q == 0 || p.num_seqs == 0) return VERIFY_OK;
    if (!k_new || !v_new || !block_tables || !seq_lens || !q_start || !k_cache || !v_cache)
        return VERIFY_EINVAL;
    if (p.num_kv_heads > 65535) return VERIFY_EUNSUPPORTED;  // grid y
    const dim3 grid((unsigned)p.num_seqs, (unsigned)p.num_kv_heads);
#define AVERIFY_APPEND(T, D)                                                                       \
    hipLaunchKernelGGL((attn_kv_append<T, D>), grid, dim3(kAppendThreads), 0, stream, p.num_seqs,    \
                       p.num_kv_heads,                                                             \
                       p.max_blocks_per_seq, p.num_blocks, static_cast<const T*>(k_new),          \
                       static_cast<const T*>(v_new), block_tables, seq_lens, q_start,             \
                       static_cast<T*>(k_cache), static_cast<T*>(v_cache))
    if (p.dtype == VERIFY_BF16) {
        if (p.head_dim == 128) AVERIFY_APPEND(uint16_t, 128);
        else AVERIFY_APPEND(uint16_t, 64);
    } else {
        if (p.head_dim == 128) AVERIFY_APPEND(float, 128);
        else AVERIFY_APPEND(float, 64);
    }
#undef AVERIFY_APPEND
    return check_launch();
}
