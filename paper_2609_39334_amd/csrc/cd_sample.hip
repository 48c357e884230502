// Branching sampler of computation deduplication (Sec. 4.2).  A sequence with potential size n
// stands for n identical candidates; one decode step over it yields one row of logits, from which
// n tokens are drawn as independent trials and grouped: one child per distinct token, whose
// potential is the group's size.  The distribution is the temperature softmax of the row (Sec. 2.1).
//
// One workgroup per row, so rows of every potential size run in one launch.  A draw is the inverse
// CDF at the caller's uniform u: the first token (in token order) whose cumulative weight exceeds
// u * Z.  The row is read once, in tiles of 4,096 logits, one wave per tile: lane l owns the 16
// contiguous logits [16l, 16l + 16) of each of the tile's four 1,024-logit parts.  (Rows of up to 16,384
// logits take tiles of one part, so that more waves share them.)  The kernel's CDF is defined by its own
// fp32 sums:
//   tile i: base b_i = the tile's maximum, w_j = exp2((l_j - b_i) * log2(e) / T);
//   s_l = w over lane l's 16 logits of a part, added in token order; the part's total is the sum of s_l
//   over the lanes as a balanced binary tree; the part totals added in order give the tile total
//   T_i and each part's start;
//   with M the row maximum and f_i = exp2((b_i - M) * log2(e) / T), the tile prefixes
//   P_0 = 0, P_{i+1} = P_i + f_i T_i, one tile at a time, and Z = P_{n_tiles}.
//   Lane l of a part starts at F_l = P_i + f_i (part start + lanes before it, by a fixed shuffle
//   pattern), and its token j is at F_l + f_i (w of its logits up to j, in token order).
// A draw finds the tile with P_i <= u Z < P_{i+1} and the part whose start is the last at or below
// u Z; one wave reloads that part and repeats the same arithmetic; of the lanes that own a weight, the
// last that starts at or below u Z scans its 16 logits, and a target its rounding leaves past its last
// token goes to its last token with a weight.  Zero weights (logit -inf, or so low that exp2 gives 0) are
// never drawn.  Grouping: each draw that is the first of its token counts the token's draws and writes it
// at its rank among the distinct tokens, so groups come out in ascending token order.
//
// What bounds it: reading the logits.  A wave works on its own tile, so nothing waits at a barrier
// until the row is read, and a workgroup of W waves keeps W tiles (16 KB each) in flight.  The tile
// is loaded in contiguous 1-KB runs and handed to its owning lanes through LDS: read in place (64
// contiguous bytes per lane), every 128-byte line is touched by four loads.  On 1,627 rows of
// 151,936 logits: 199.6 us with one 256-thread workgroup per row and barriers in every tile, 173 us
// with a wave per tile, 155 us (6.4 TB/s) with contiguous non-temporal loads.  On 16 such rows: 52.9,
// 16.1 and 15.2 us (the last without the non-temporal hint, see tkv_cd_sample).
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdint>

#include "internal.h"

namespace {

constexpr int kPerLane = 16;                  // contiguous logits per lane and part
constexpr int kPart = 64 * kPerLane;          // 1,024 logits
constexpr int kMaxVocab = 512 * 4 * kPart;    // 2,097,152
constexpr int kMaxPotential = 1024;           // draws of one row (grouped in LDS)

typedef float f32x4_t __attribute__((ext_vector_type(4), aligned(4)));  // rows need not start 16-byte aligned

// Orders a wave's LDS writes before its lanes' later reads and the reverse (a wave's LDS operations run
// in program order: this only keeps the compiler from moving them).
__device__ __forceinline__ void lanes_agree() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The 16 logits of each part that this lane owns, of a tile that lies inside the vocabulary: loaded in
// 1-KB runs (lane l takes the l-th 16 bytes of a run) and passed through the wave's 4 KB of LDS, a
// part at a time; chunk q of a part sits at q ^ ((q / 16) % 4), so that neither the writes (64
// consecutive chunks) nor the reads (chunks 4l + e) meet in a bank.  NT: non-temporal loads.
template <int PARTS, bool NT>
__device__ __forceinline__ void load_tile(const float* __restrict__ tile, int lane, float4* __restrict__ lds,
                                          float (&x)[PARTS][kPerLane]) {
    const f32x4_t* r4 = reinterpret_cast<const f32x4_t*>(tile) + lane;
    f32x4_t g[PARTS][4];
#pragma unroll
    for (int p = 0; p < PARTS; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            g[p][j] = NT ? __builtin_nontemporal_load(r4 + (p * kPart / 4 + 64 * j)) : r4[p * kPart / 4 + 64 * j];
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = 64 * j + lane;
            lds[q ^ ((q >> 4) & 3)] = make_float4(g[p][j][0], g[p][j][1], g[p][j][2], g[p][j][3]);
        }
        lanes_agree();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float4 v = lds[(4 * lane + e) ^ ((lane >> 2) & 3)];
            x[p][4 * e] = v.x;
            x[p][4 * e + 1] = v.y;
            x[p][4 * e + 2] = v.z;
            x[p][4 * e + 3] = v.w;
        }
        lanes_agree();
    }
}

// This lane's 16 logits of the part that starts at token a0 (positions past the vocabulary read as
// -inf).
__device__ __forceinline__ void load16(const float* __restrict__ row, int vocab, int a0, int lane, float (&x)[kPerLane]) {
    const int a = a0 + lane * kPerLane;
    if (a + kPerLane <= vocab) {
        const f32x4_t* r4 = reinterpret_cast<const f32x4_t*>(row + a);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const f32x4_t v = r4[k];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[4 * k + e] = v[e];
        }
    } else {
#pragma unroll
        for (int k = 0; k < kPerLane; ++k) x[k] = a + k < vocab ? row[a + k] : -INFINITY;
    }
}

// v of the lane whose index differs in bit 0, 1, 2 or 3 -- for values that already agree over the
// lower bits, where a mirror within 8 or 16 lanes reaches the right group.
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Balanced-tree reduction over the 64 lanes (every lane gets it): pairs at distance 1, 2, ..., 32.
template <class Op>
__device__ __forceinline__ float wave_tree(float v, Op op) {
    v = op(v, dpp<0xb1>(v));   // quad_perm [1, 0, 3, 2]
    v = op(v, dpp<0x4e>(v));   // quad_perm [2, 3, 0, 1]
    v = op(v, dpp<0x141>(v));  // row_half_mirror
    v = op(v, dpp<0x140>(v));  // row_mirror
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Inclusive scan of v over the 64 lanes (fixed pattern: lane l adds lane l - 2^k when it exists; lane
// 63 holds the balanced tree's sum).
__device__ __forceinline__ float wave_scan(float v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float u = __shfl_up(v, o);
        if (lane >= o) v += u;
    }
    return v;
}

// Sum of this lane's weights in token order, each w = exp2((x - b) * c).
__device__ __forceinline__ float lane_sum(const float (&x)[kPerLane], float b, float c) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < kPerLane; ++k) s += __builtin_amdgcn_exp2f((x[k] - b) * c);
    return s;
}

// W waves per row, PARTS per tile, NT: non-temporal loads, TILES: the most tiles a row may have.  Four waves
// are for many rows, which want as many workgroups on a CU as fit: six with four parts (two registers go to
// scratch for that), eight with one.
template <int W, int PARTS, bool NT, int TILES>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(PARTS == 1 ? 8 : W == 4 ? 6 : 4))) void cd_sample(
    const float* __restrict__ logits, int vocab, float c, const float* __restrict__ uniform,
    const int32_t* __restrict__ draw_off, int32_t n_draws, int32_t* __restrict__ out_tok, int32_t* __restrict__ out_cnt,
    int32_t* __restrict__ n_groups) {
    constexpr int kTile = PARTS * kPart;
    __shared__ float base[TILES];             // b_i
    __shared__ float part[TILES][PARTS];      // the starts of tile i's parts past the first, and its total
    __shared__ float P[TILES + 1];            // tile prefixes
    __shared__ float row_max;
    __shared__ int32_t wcnt[W];
    // each wave's 4 KB for load_tile; once the row is read, the draws
    __shared__ float4 shared_mem[(W < 4 ? 4 : W) * kPart / 4];
    static_assert(sizeof(shared_mem) >= 16 * kMaxPotential, "room for the draws");
    float* target = reinterpret_cast<float*>(shared_mem);
    int32_t* tok = reinterpret_cast<int32_t*>(shared_mem) + kMaxPotential;
    int32_t* first = tok + kMaxPotential;
    int32_t* tile_of = first + kMaxPotential;
    const int r = blockIdx.x, t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const float* row = logits + static_cast<size_t>(r) * vocab;
    const int off = draw_off[r], n = draw_off[r + 1] - off;
    const int n_tiles = (vocab + kTile - 1) / kTile;
    // a row whose draws fall outside the caller's arrays (offsets are device data the host cannot
    // check), or too many of them, is refused before anything of it is read or written
    if (n < 0 || off < 0 || static_cast<int64_t>(off) + n > n_draws || n > kMaxPotential || n_tiles > TILES) {
        if (t == 0) n_groups[r] = -1;
        return;
    }
    const auto add = [](float a, float b) { return a + b; };
    const auto max2 = [](float a, float b) { return fmaxf(a, b); };

    // one pass over the row: per tile its maximum, its parts' starts and its total over that base
    for (int i = w; i < n_tiles; i += W) {
        float x[PARTS][kPerLane];
        if ((i + 1) * kTile <= vocab) {
            load_tile<PARTS, NT>(row + i * kTile, lane, shared_mem + w * (kPart / 4), x);
        } else {
#pragma unroll
            for (int p = 0; p < PARTS; ++p) load16(row, vocab, i * kTile + p * kPart, lane, x[p]);
        }
        float m = x[0][0];
#pragma unroll
        for (int p = 0; p < PARTS; ++p)
#pragma unroll
            for (int k = 0; k < kPerLane; ++k) m = fmaxf(m, x[p][k]);
        const float b = wave_tree(m, max2);
        float s[PARTS];
#pragma unroll
        for (int p = 0; p < PARTS; ++p) s[p] = wave_tree(b == -INFINITY ? 0.f : lane_sum(x[p], b, c), add);
        if (lane == 0) {
            base[i] = b;
            float sum = s[0];
            part[i][0] = sum;
#pragma unroll
            for (int p = 1; p < PARTS; ++p) part[i][p] = sum += s[p];
        }
    }
    __syncthreads();
    if (w == 0) {
        float mx = -INFINITY;
        for (int i = lane; i < n_tiles; i += 64) mx = fmaxf(mx, base[i]);
        mx = wave_tree(mx, max2);
        float sum = 0.f;
        for (int i0 = 0; i0 < n_tiles; i0 += 64) {
            const int i = i0 + lane;
            const float f = i < n_tiles && base[i] != -INFINITY ? __builtin_amdgcn_exp2f((base[i] - mx) * c) : 0.f;
            const float total = i < n_tiles ? part[i][PARTS - 1] : 0.f;
            float mine = 0.f;  // P of this lane's tile
            for (int k = 0; k < min(64, n_tiles - i0); ++k) {
                if (lane == k) mine = sum;
                sum = fmaf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), k)),
                           __int_as_float(__builtin_amdgcn_readlane(__float_as_int(total), k)), sum);
            }
            if (i < n_tiles) P[i] = mine;
        }
        if (lane == 0) {
            P[n_tiles] = sum;
            row_max = mx;
        }
    }
    __syncthreads();
    const float mx = row_max;
    if (mx == -INFINITY) {  // no finite logit: no distribution
        if (t == 0) n_groups[r] = -1;
        return;
    }
    const float Z = P[n_tiles];

    // each draw's target and tile (first tile with P[i + 1] > target; n_tiles if u Z rounded up to Z)
    for (int k = t; k < n; k += 64 * W) {
        const float tg = uniform[off + k] * Z;
        int lo = 0, hi = n_tiles;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (P[mid + 1] > tg) hi = mid; else lo = mid + 1;
        }
        target[k] = tg;
        tile_of[k] = lo;
        tok[k] = -1;
    }
    __syncthreads();

    // resolve the draws, one wave each: reload the part that holds the target and repeat its arithmetic
    // (once for a run of draws in one part)
    int held = -1;  // the part whose logits and starts are in x and start
    float x[kPerLane], start = 0.f;
    uint64_t weighted = 0;  // the lanes with a weight in it
    for (int k = w; k < n; k += W) {
        const int i = __builtin_amdgcn_readfirstlane(tile_of[k]);
        if (i >= n_tiles) continue;
        const float tg = target[k], b = base[i], p0 = P[i];
        const float f = __builtin_amdgcn_exp2f((b - mx) * c);
        // (the sums that P is made of, so the part has a weight: behind one without, the next starts no later)
        int pi = 0;
#pragma unroll
        for (int p = 1; p < PARTS; ++p)
            if (fmaf(f, part[i][p - 1], p0) <= tg) pi = p;
        pi = __builtin_amdgcn_readfirstlane(pi);
        const int a0 = i * kTile + pi * kPart;
        if (a0 != held) {
            held = a0;
            load16(row, vocab, a0, lane, x);
            const float sum = lane_sum(x, b, c);
            weighted = __builtin_amdgcn_ballot_w64(sum > 0.f);
            const float incl = wave_scan(sum, lane);
            float excl = __shfl_up(incl, 1);
            if (lane == 0) excl = 0.f;
            start = p0 + f * ((pi == 0 ? 0.f : part[i][pi - 1]) + excl);
        }
        // (the scan's sums do not rise evenly: lanes behind the last weight may start at or below the target)
        const uint64_t below = weighted & __builtin_amdgcn_ballot_w64(start <= tg);
        if (lane == (below ? 63 - __builtin_clzll(below) : __builtin_ctzll(weighted | uint64_t{1} << 63))) {
            const int a = a0 + lane * kPerLane;
            int pick = -1, last = -1;
            float acc = 0.f;
#pragma unroll
            for (int q = 0; q < kPerLane; ++q) {
                const float wq = __builtin_amdgcn_exp2f((x[q] - b) * c);
                acc += wq;
                if (wq > 0.f) last = a + q;
                if (pick < 0 && wq > 0.f && start + f * acc > tg) pick = a + q;
            }
            tok[k] = pick >= 0 ? pick : last;
        }
    }
    __syncthreads();
    // targets past every tile (u Z = Z, for u = 1): the row's last token with a weight
    for (int k = t; k < n; k += 64 * W) {
        if (tok[k] >= 0) continue;
        int j = vocab - 1;
        while (j > 0 && __builtin_amdgcn_exp2f((row[j] - mx) * c) == 0.f) --j;
        tok[k] = j;
    }
    __syncthreads();

    // group: first occurrences count their token's draws and go to their rank among distinct tokens
    for (int k = t; k < n; k += 64 * W) {
        bool is_first = true;
        for (int j = 0; j < k && is_first; ++j) is_first = tok[j] != tok[k];
        first[k] = is_first ? 1 : 0;
    }
    __syncthreads();
    int mine = 0;
    for (int k = t; k < n; k += 64 * W) {
        if (!first[k]) continue;
        int cnt = 0, rank = 0;
        for (int j = 0; j < n; ++j) {
            cnt += tok[j] == tok[k];
            rank += first[j] && tok[j] < tok[k];
        }
        out_tok[off + rank] = tok[k];
        out_cnt[off + rank] = cnt;
        ++mine;
    }
    for (int o = 32; o > 0; o >>= 1) mine += __shfl_xor(mine, o);
    if (lane == 0) wcnt[w] = mine;
    __syncthreads();
    if (t == 0) {
        int groups = 0;
        for (int k = 0; k < W; ++k) groups += wcnt[k];
        n_groups[r] = groups;
    }
}

}  // namespace

TKV_EXPORT int tkv_cd_sample(int32_t n_rows, int32_t vocab, float temperature, int32_t max_potential,
                             const float* d_logits, const float* d_uniform, const int32_t* d_draw_off,
                             int32_t n_draws, int32_t* d_token, int32_t* d_count, int32_t* d_n_groups, void* stream) {
    tkv::clear_error();
    if (n_rows < 0 || vocab < 1) return tkv::set_error(TKV_EINVAL, "tkv_cd_sample: n_rows %d, vocab %d", n_rows, vocab);
    if (vocab > kMaxVocab) return tkv::set_error(TKV_EINVAL, "tkv_cd_sample: vocabulary %d exceeds %d", vocab, kMaxVocab);
    if (!(temperature > 0.f) || !std::isfinite(temperature))
        return tkv::set_error(TKV_EINVAL, "tkv_cd_sample: temperature must be positive and finite");
    if (max_potential < 0 || max_potential > kMaxPotential)
        return tkv::set_error(TKV_EINVAL, "tkv_cd_sample: potential up to %d per row (got %d)", kMaxPotential, max_potential);
    if (n_draws < 0) return tkv::set_error(TKV_EINVAL, "tkv_cd_sample: n_draws = %d < 0", n_draws);
    if (n_rows == 0) return TKV_OK;
    if (!d_logits || !d_draw_off || !d_n_groups || (n_draws > 0 && (!d_uniform || !d_token || !d_count)))
        return tkv::set_error(TKV_EINVAL, "tkv_cd_sample: NULL pointer");
    const float c = 1.4426950408889634f / temperature;
    const hipStream_t st = static_cast<hipStream_t>(stream);
    auto launch = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(n_rows)), dim3(static_cast<unsigned>(64 * waves)), 0, st,
                           d_logits, vocab, c, d_uniform, d_draw_off, n_draws, d_token, d_count, d_n_groups);
    };
    // Logits that the 256 MB Infinity Cache cannot hold are read with the non-temporal hint (155 against
    // 171 us on 1,627 rows of 151,936); smaller ones may still sit there, as the head's product left
    // them, and the hint would pass that by (19.2 against 15.2 us on 16 rows, 19.9 against 16.0 on 64).
    // Up to 256 rows each row has a CU to itself and takes 16 waves (15.4 against 18.4 us with 8 on 16
    // rows of 151,936).  Beyond that several rows share a CU, and waves without a tile of their own only
    // hold up the next workgroup: 4 waves up to 65,536 logits (1,000 rows of 50,257 36.8 us, 38.2 with 8, 50.2
    // with 16), 2 for more rows of up to 32,768 (5,000 rows of 17,000 63 us, 73 with 4, 110 with 8) while
    // their draws are few, 8 on longer rows (171 against 175 us with 4 at 151,936) and past the cache from
    // 32,768 on (1,600 rows of 50,257 58.8 us, 61.3 with 4).
    // Rows of up to 16,384 logits take tiles of one part: 300 rows of 600 6.1 us, 8.3 with four parts;
    // 20,000 rows of 4,096 70 us, 94; 120,000 rows of 600 353 us, 654; 256 rows of 8,191 on 16 waves 6.3 us,
    // 6.9.  Many draws a row want more waves (1,000 rows of 4,096 with 200 draws: 116 us on 8, 128 on 4).
    const bool past = static_cast<int64_t>(n_rows) * vocab > (int64_t{256} << 20) / 4;
    if (vocab <= 16 * kPart) {
        if (n_rows <= 256)
            launch(cd_sample<16, 1, false, 16>, 16);
        else if (max_potential > 64)
            launch(cd_sample<8, 1, false, 16>, 8);
        else if (past)
            launch(cd_sample<4, 1, true, 16>, 4);
        else
            launch(cd_sample<4, 1, false, 16>, 4);
    } else if (n_rows > 256 && vocab <= (past ? 8 : 16) * 4 * kPart) {
        if (n_rows > 1024 && vocab <= 8 * 4 * kPart && max_potential <= 8) {
            if (past)
                launch(cd_sample<2, 4, true, 8>, 2);
            else
                launch(cd_sample<2, 4, false, 8>, 2);
        } else if (past) {
            launch(cd_sample<4, 4, true, 16>, 4);
        } else {
            launch(cd_sample<4, 4, false, 16>, 4);
        }
    } else if (past) {
        launch(cd_sample<8, 4, true, 512>, 8);
    } else if (n_rows <= 256) {
        launch(cd_sample<16, 4, false, 512>, 16);
    } else {
        launch(cd_sample<8, 4, false, 512>, 8);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return tkv::set_error(TKV_EHIP, "tkv_cd_sample launch: %s", hipGetErrorString(e));
    return TKV_OK;
}
