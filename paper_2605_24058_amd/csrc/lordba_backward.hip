// Backward pass of the LoRDBA adapter branch for MI355X (gfx950, wave64, MFMA), as training needs it (Sec. 3.2 "Forward
// and backward pass"; smooth-sign straight-through factor of Eq. (smoothsign); Alg. QAT-LoRDBA).
//
// Forward (Eq. (lordba-fwd)):  w = x D_alpha, t = w B1, u = t D_beta, v = u B2, y = y_base + v D_gamma, with S_A = B1^T
// [r, d_in], S_B = B2^T [d_out, r].  For an upstream gradient g = dL/dy:
//
//   du = (g D_gamma) B2^T          dt = du D_beta           dx = dx_base + (dt B1^T) D_alpha
//   Q  = dt^T x   [r, d_in]        P  = u^T g   [r, d_out]  (contractions over the token rows)
//   d_alpha_i = sum_k S_A[k,i] Q[k,i]       dS_A[k,i] = alpha_i Q[k,i]
//   d_gamma_j = sum_k S_B[j,k] P[k,j]       dS_B[j,k] = gamma_j P[k,j]
//   d_beta_k  = sum_t du[t,k] t[t,k]
//   d_latent  = dS * kappa (1 - tanh^2(kappa latent))                                    (Eq. (smoothsign))
//
// Kernels, all on the caller's stream, no host synchronisation, every buffer beyond inputs and outputs in the caller's
// workspace:
//   dx      The forward kernel itself on the transposed adapter: DeltaW^T has the form of Eq. (lordba) with the carriers
//           transposed and alpha, gamma exchanged.  Its rank-r intermediate is du, which it also writes out.
//   t       The forward kernel on x, stopped after its rank-r intermediate t (skipped when the caller kept t from the
//           training forward pass, lordba_forward_save_t).  With several envelopes both calls produce the intermediates of
//           all envelopes at once; wgrad and finish then run once per envelope.
//   wgrad   Q and P: MFMA with the token rows as contraction index.  A lane reads 8 token rows x 8 columns of x (or g)
//           with row-contiguous 16-byte loads and transposes its 8 x 8 block in registers (v_perm_b32); MFMA e of a step
//           takes column 8 m + e from lane group m.  du (or t) enters as fp16 hi + lo after a power-of-two scaling per rank that
//           follows the largest entry seen so far, and beta behind the sums (element-aligned tensors: beta du and beta t enter, as
//           hi + lo + rest).  Token ranges are split over waves and workgroups; partial sums are reduced in a fixed order.  From
//           two rank blocks on and with enough to stream, a second kernel takes the tokens through LDS (see there).
//   finish  sums the partials, applies the carrier signs, the scales and the smooth-sign factor; and d_beta.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "lordba.h"
#include "lordba_dev_util.h"
#include "lordba_rows.h"

namespace {

constexpr int kWgradWaves = 4;        // waves per workgroup of the wgrad kernel, each with its own token range (8 on short batches)
// Workgroups the wgrad grid aims at: two per CU once the token ranges are long (measured 3-4 % faster from T = 4096 on),
// one per CU below that, where a second one only doubles the partial sums the finish kernel has to read.
constexpr int kWgradTargetWgsLong = 512, kWgradTargetWgsShort = 256;
// 32-row steps a wave of the wgrad kernel keeps in flight: one.  Deeper requests per wave
// were slower wherever they were tried (four steps against one: 4 to 5 % of the whole call at T = 8192, 1 to 6 % below 4096);
// a kernel that only reads the same column stripes shows the same (5120 columns, 8192 rows, 240 workgroups: 4.4 TB/s with
// four steps in flight per wave, 5.9 with one or two): a wave that requests 128 rows at a time spreads its requests over
// more DRAM pages than one that walks 32 rows at a time.
constexpr int kWgradGroup = 1;
constexpr int kShortBatch = 4096;     // token rows from which a batch counts as long

struct BwdPlan {
    int rp;          // ranks padded to a multiple of 16
    int t_pad;       // token rows padded to a multiple of 128 (whole groups of steps of the wgrad kernel, whole 16-byte pieces of t and du)
    int nbx, nbg;    // 128-column blocks of d_in and of d_out
    int dcols;       // columns of one partial-sum plane: (nbx + nbg) * 128
    int tw;          // token rows per wave of the wgrad kernel (a multiple of 32, or of 64: see group_rows)
    int splits;      // workgroups along the token axis of the wgrad kernel
    int waves;       // waves per workgroup of the wgrad kernel: 4, or 8 on short batches with one rank block (see make_plan)
    // workspace layout, in 4-byte words
    size_t off_t, off_du, off_part, off_rank, words;
};

// ell_fused: envelopes whose partial sums the wgrad kernel holds at once (1: one envelope per wgrad / finish pass).
BwdPlan make_plan(int64_t T, int64_t d_in, int64_t d_out, int64_t r, int64_t ell_fused = 1) {
    BwdPlan p;
    p.rp = static_cast<int>((r + 15) / 16 * 16);
    p.t_pad = static_cast<int>((T + 127) / 128 * 128);
    p.t_pad = p.t_pad < 128 ? 128 : p.t_pad;  // T == 0 still yields a well-formed (unused) plan
    p.nbx = static_cast<int>((d_in + 127) / 128);
    p.nbg = static_cast<int>((d_out + 127) / 128);
    p.dcols = (p.nbx + p.nbg) * 128;
    // Below 4096 token rows a wave of a 4-wave workgroup would have little to overlap with: such batches run 8 waves (two
    // per SIMD); from two rank blocks on their workgroups share a compute unit instead (see launch_all).
    p.waves = T < kShortBatch && p.rp * ell_fused <= 16 ? 2 * kWgradWaves : kWgradWaves;
    // (beyond 2048 rows with three or four rank blocks: token ranges of 64 rows at a time, so that the plan, and with it the shapes that fit
    // the array of lordba_backward_noalloc, is the one it was when such a workgroup took two steps at a time)
    const int group_rows = T > 2048 && p.rp * ell_fused > 32 ? 64 : 32 * kWgradGroup;
    const int groups = p.t_pad / group_rows;  // a wave takes whole groups of steps (t_pad is a multiple of 128)
    const int target = T >= kShortBatch ? kWgradTargetWgsLong : kWgradTargetWgsShort;
    int splits = target / (p.nbx + p.nbg);   // rounded down: a grid just above the target would start another round
    const int max_splits = (groups + p.waves - 1) / p.waves;  // at least one group per wave
    splits = splits > max_splits ? max_splits : splits;
    splits = splits < 1 ? 1 : splits;
    const int groups_per_wave = (groups + splits * p.waves - 1) / (splits * p.waves);
    p.tw = groups_per_wave * group_rows;
    p.splits = (groups + groups_per_wave * p.waves - 1) / (groups_per_wave * p.waves);
    // t and du: one [r, t_pad] block per envelope, room for the largest envelope count
    p.off_t = 0;
    p.off_du = p.off_t + static_cast<size_t>(LORDBA_MAX_ENVELOPES) * p.rp * p.t_pad;
    p.off_part = p.off_du + static_cast<size_t>(LORDBA_MAX_ENVELOPES) * p.rp * p.t_pad;
    // one word per rank and token range for d_s_rank: arrivals and, one part fewer than there are token ranges, the sums of its parts
    p.off_rank = p.off_part + static_cast<size_t>(p.splits) * p.rp * ell_fused * p.dcols;
    p.words = p.off_rank + static_cast<size_t>(p.splits) * p.rp * ell_fused;
    return p;
}

struct BwdArgs {
    const _Float16* x;
    const _Float16* g;
    const uint32_t* pA;    // S_A   [r, d_in]
    const uint32_t* pBt;   // S_B^T [r, d_out]
    const _Float16* s_in;
    const _Float16* s_rank;
    const _Float16* s_out;
    const float* latA;     // [r, d_in]
    const float* latB;     // [d_out, r]
    float kappa;
    float* d_s_in;
    float* d_s_rank;
    float* d_s_out;
    float* d_latA;
    float* d_latB;
    const float* tT;       // t,  rank-major: tT[k * t_stride + token], defined for k < r, token < T
    const float* duT;      // du, rank-major: duT[k * du_stride + token]
    float* part;           // [splits, ell, rp, dcols]
    int T, d_in, d_out, r;
    int rp, t_pad, t_stride, du_stride, nbx, nbg, dcols, tw, splits, waves;
    float* rank_sums;      // [1 + rank_parts, ell, rp]: arrivals (as whole numbers), then the parts' sums of d_s_rank (rank_parts > 1)
    int rank_parts, rank_tokens;   // workgroups per rank of d_s_rank, tokens of each (but the last)
    int accumulate;        // latent gradients are added to what the arrays hold (second and later envelopes, one pass each)
    // Envelopes held at once (Eq. (lordba): the carriers are shared, so Q and P of all envelopes contract the same x and g
    // with different small operands).  s_in, s_rank, s_out and the scale gradients then have ell rows, tT and duT one
    // [r, stride] block per envelope, and the wgrad kernel's rank blocks are the ell * rp / 16 blocks of all envelopes.
    int ell;
    int any;               // widths that are no multiples of 32, or tensors aligned to their elements only
};

// The scaling of a rank's entries (see the wgrad kernel): cur_e follows the largest entry seen so far, of the eight that each of the four lane
// groups brings.  Returns the factor (a power of two) by which what has been accumulated has to be rescaled.
__device__ __forceinline__ float follow_largest(const float (&v)[8], int& cur_e) {
    float m = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fabsf(v[2]));
    m = fmaxf(fmaxf(m, fabsf(v[3])), fabsf(v[4]));
    m = fmaxf(fmaxf(m, fabsf(v[5])), fabsf(v[6]));
    m = max_of_lane_groups(fmaxf(m, fabsf(v[7])));
    int e = static_cast<int>((__float_as_uint(m) >> 23) & 0xffu);
    e = e > 254 ? 254 : e;
    const int sh = cur_e - e;
    cur_e = e > cur_e ? e : cur_e;
    return sh >= 0 ? 1.f : (sh < -126 ? 0.f : __uint_as_float(static_cast<uint32_t>(127 + sh) << 23));
}
// v mul as fp16 hi + lo, one rounding each (mixed-precision multiply-adds, two instructions per entry)
__device__ __forceinline__ void split_scaled(const float (&v)[8], float mul, u4& hi, u4& lo) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        h2 h, l;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            h[j] = static_cast<_Float16>(__builtin_fmaf(v[2 * w + j], mul, 0.f));
            l[j] = static_cast<_Float16>(__builtin_fmaf(v[2 * w + j], mul, -static_cast<float>(h[j])));
        }
        hi[w] = __builtin_bit_cast(uint32_t, h);
        lo[w] = __builtin_bit_cast(uint32_t, l);
    }
}

__global__ void bwd_zero_kernel(float* p, int64_t n) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.f;
}

// No rank has been added up yet: by one wave of the kernel before, at its start (behind everything else the look at the arguments is a trip to
// memory that every wave 0 ends with: 0.1 us of a call of 29.7 at 2048 x 4096 x 4096, r = 16).
__device__ __forceinline__ void clear_rank_arrivals(const BwdArgs& a, int lane) {
    if (a.rank_parts > 1 && blockIdx.x == 0 && blockIdx.y == 0 && lane < a.ell * a.rp) reinterpret_cast<uint32_t*>(a.rank_sums)[lane] = 0u;
}

// ----------------------------------------------------------------------------------------- wgrad kernel ----
// Workgroup (cb, s): column block cb of x (cb < nbx: Q, with du) or of g (P, with t), token rows [s * W tw, (s+1) * W tw),
// one range of tw rows per wave.  One step = 32 token rows x 128 columns.
// G steps are in flight per wave: the loads of a group are issued without any condition (past the end of the wave's range
// they re-read valid addresses and are not used), so that every wait counts exactly the loads issued after the one it
// needs; the last group is consumed without issuing anything.
// ANY: any widths from 8 columns on, accesses without an alignment; a last group of 8 columns that reaches past the row is read 8
// columns from its end and moved into place (columns past the end are zeros).  Infinities propagate by IEEE rules, as in the general
// kernel.
template <int RB, int G, int W, int Z, bool ANY>
__global__ __launch_bounds__(W * 64) void lordba_bwd_wgrad_kernel(BwdArgs a) {
    static_assert(W == 4 || W == 8, "the final sums are dealt to 4 or 8 waves");
    __shared__ __align__(16) float red[W][8][64][4];
    // The wave index as a scalar: everything that depends on it (how many steps) then branches on scalar conditions.
    // MFMA instructions ignore the EXEC mask, so they must never sit under a vector-predicated branch.
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, q = lane >> 4;
    if (wave == 0) clear_rank_arrivals(a, lane);
    const int rbe = a.rp >> 4, blocks = a.ell * rbe;  // rank blocks per envelope, and in all
    int cb = blockIdx.x, rb0 = 0;   // column block, first rank block
    if constexpr (Z > 1) {
        // workgroups are dealt to the 8 XCDs in turn: the Z that read the same x (or g) are 8 apart, on one XCD
        rb0 = (cb >> 3) % Z * RB;
        cb = (cb / (8 * Z)) * 8 + (cb & 7);
        if (cb >= a.nbx + a.nbg) return;   // (the whole workgroup, before any barrier)
    }
    const int tk_begin = (static_cast<int>(blockIdx.y) * W + wave) * a.tw;
    int tk_end = tk_begin + a.tw;
    tk_end = tk_end < a.t_pad ? tk_end : a.t_pad;

    const bool is_x = cb < a.nbx;
    const int cc = is_x ? cb : cb - a.nbx;
    const int d = is_x ? a.d_in : a.d_out;
    const _Float16* src = is_x ? a.x : a.g;
    const float* small = is_x ? a.duT : a.tT;   // du meets x, t meets g (ANY: times beta; otherwise beta comes in at the end)
    const int sstride = is_x ? a.du_stride : a.t_stride;

    float beta[RB];
    int row_of[RB];  // the lane's row in the small arrays: envelope * r + rank, clamped to a rank that exists (its values are then masked)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {   // block b: envelope b / (rp / 16), ranks 16 (b % (rp / 16)) ..  (past the last block: it again)
        const int b = rb0 + rb < blocks ? rb0 + rb : blocks - 1, en = b / rbe, rk = (b - en * rbe) * 16 + li;
        row_of[rb] = en * a.r + (rk < a.r ? rk : a.r - 1);
        beta[rb] = rk < a.r ? static_cast<float>(a.s_rank[row_of[rb]]) : ANY ? 0.f : 1.f;   // (a padded rank's sums are never used)
    }
    bool silent = false;   // a rank without scale among this wave's: it adds nothing, whatever its entries are (!ANY)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) silent |= __builtin_amdgcn_ballot_w64(beta[rb] == 0.f) != 0ull;
    int col = cc * 128 + li * 8;
    const int back = ANY && col > d - 8 ? col - (d - 8) : 0;   // columns that a ragged group was moved back by
    col = ANY ? col - back : (col < d ? col : d - 8);  // past the end: a valid column group is re-read, its sums are never used

    f4 acc[RB][8];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[rb][e] = f4{0.f, 0.f, 0.f, 0.f};
    }
    // Power-of-two scaling per rank: 2^(140 - cur_e) brings an entry with biased exponent cur_e to [2^13, 2^14), so that
    // hi + lo (two fp16) keep 22 bits of it.  cur_e follows the largest entry of the rank seen so far, group by group; when
    // it grows, what has been accumulated is rescaled.  Entries far below the largest lose bits that do not matter to the sum.
    // ANY: hi + lo + rest keep the 24 bits that the general kernel multiplies with (of entries down to 2^-14 of the largest): it took
    // these calls before.  Error against 64 bits on 40 odd shapes of 1 to 600 rows, relative to the general kernel's: 0.70 to 0.74
    // (geometric mean of each gradient); with hi + lo alone 0.75 to 0.78, but up to 1.13 below 25 rows.  The third product and the
    // care for infinities cost 1 to 3 % of a call (300 x 1000 -> 3001, r = 12 17.1 -> 17.4 us; 600 x 4728 -> 11055, r = 32 37.2 -> 37.7).
    int cur_e[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) cur_e[rb] = 14;

    u4 xb[G][8];         // x (or g): step i of the group, 8 token rows x 8 columns per lane
    u4 sb[G][RB][2];     // du (or t): 8 tokens of the lane's rank per step, fp32
    constexpr int NS = ANY ? 3 : 2;
    u4 hl[G][RB][NS];    // the same as fp16 hi and lo operands, scaled (ANY: and what is left of the 24 bits)
    auto issue_x = [&](int i, int tk) {
        tk = tk < a.t_pad - 32 ? tk : a.t_pad - 32;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            int row = tk + 8 * q + e;
            row = row < a.T ? row : a.T - 1;  // rows past T meet du = t = 0
            const _Float16* p = src + static_cast<size_t>(row) * d + col;
            xb[i][e] = ANY ? load16_any_stream(p) : load16_stream(p);
        }
    };
    auto issue_small = [&](int tk0) {  // all G steps of the group that starts at token tk0
#pragma unroll
        for (int i = 0; i < G; ++i) {
            int tk = tk0 + 32 * i;
            tk = tk < a.t_pad - 32 ? tk : a.t_pad - 32;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                // 32 bytes inside the row's t_pad entries; the array is defined for token < T only, the rest is masked
                const float* p = small + static_cast<size_t>(row_of[rb]) * sstride;
                const int tok = tk + 8 * q;
                if constexpr (ANY) {   // (nothing past the row's T entries is read: a kept t may end there; see convert)
                    sb[i][rb][0] = load16_word(p + row_piece(tok, a.T, row_of[rb]));
                    sb[i][rb][1] = load16_word(p + row_piece(tok + 4, a.T, row_of[rb]));
                } else {
                    sb[i][rb][0] = load16(p + tok);
                    sb[i][rb][1] = load16(p + tok + 4);
                }
            }
        }
    };
    auto convert = [&](int tk0) {  // scale of the group, then its hi / lo (/ rest) operands
        if constexpr (!ANY) {
            static_assert(G == 1, "one step at a time");
            if (silent || tk0 + 32 > a.T) {   // scalar: the last rows (entries past T are undefined)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) sb[0][rb][e >> 2][e & 3] = beta[rb] != 0.f && tk0 + 8 * q + e < a.T ? sb[0][rb][e >> 2][e & 3] : 0u;
                }
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(sb[0][rb][e >> 2][e & 3]);
                if (const float f = follow_largest(v, cur_e[rb]); __builtin_amdgcn_ballot_w64(f != 1.f) != 0ull) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[rb][e] *= f;
                }
                split_scaled(v, __uint_as_float(static_cast<uint32_t>(267 - cur_e[rb]) << 23), hl[0][rb][0], hl[0][rb][1]);
            }
        } else {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                float v[G][8];
                float m = 0.f;
#pragma unroll
                for (int i = 0; i < G; ++i) {
                    if (tk0 + 32 * i + 32 > a.T) {   // scalar: the row's last entries may have been read from its end
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const int tok = tk0 + 32 * i + 8 * q + 4 * h;
                            sb[i][rb][h] = drop_words(sb[i][rb][h], tok - row_piece(tok, a.T, row_of[rb]));
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float raw = __uint_as_float(sb[i][rb][e >> 2][e & 3]);
                        // select, not multiply: the padding rows hold undefined values
                        v[i][e] = tk0 + 32 * i + 8 * q + e < a.T ? raw * beta[rb] : 0.f;
                        m = fmaxf(m, fabsf(v[i][e]));
                    }
                }
                m = fmaxf(m, __shfl_xor(m, 16, 64));
                m = fmaxf(m, __shfl_xor(m, 32, 64));
                int e_new = static_cast<int>((__float_as_uint(m) >> 23) & 0xffu);
                e_new = e_new > 254 ? 254 : e_new;
                if (__builtin_amdgcn_ballot_w64(e_new > cur_e[rb]) != 0ull) {   // scalar branch: rare after the first group
                    const int sh = cur_e[rb] - e_new;                           // < 0 where this lane's rank grows
                    const float f = sh >= 0 ? 1.f : (sh < -126 ? 0.f : __uint_as_float(static_cast<uint32_t>(127 + sh) << 23));
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[rb][e] *= f;
                    cur_e[rb] = e_new > cur_e[rb] ? e_new : cur_e[rb];
                }
                const float mul = __uint_as_float(static_cast<uint32_t>(267 - cur_e[rb]) << 23);
#pragma unroll
                for (int i = 0; i < G; ++i) {
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        float v0 = v[i][2 * w] * mul, v1 = v[i][2 * w + 1] * mul;
#pragma unroll
                        for (int s = 0; s < NS; ++s) {
                            h2 h;
                            h[0] = static_cast<_Float16>(v0);
                            h[1] = static_cast<_Float16>(v1);
                            hl[i][rb][s][w] = __builtin_bit_cast(uint32_t, h);
                            const bool stop = s == 0;   // (nothing is left of an infinity, no inf - inf)
                            v0 = stop && !(fabsf(v0) < INFINITY) ? 0.f : v0 - static_cast<float>(h[0]);
                            v1 = stop && !(fabsf(v1) < INFINITY) ? 0.f : v1 - static_cast<float>(h[1]);
                        }
                    }
                }
            }
        }
    };
    auto consume_x = [&](int i, int tk) {
        if constexpr (ANY) {
            if (cc * 128 + 128 > d) {   // scalar: the last column block
#pragma unroll
                for (int e = 0; e < 8; ++e) xb[i][e] = drop_halves(xb[i][e], back);
            }
            if (tk + 32 > a.T) {        // scalar: the last rows (they repeat row T - 1, which may hold infinities)
#pragma unroll
                for (int e = 0; e < 8; ++e) xb[i][e] = tk + 8 * q + e < a.T ? xb[i][e] : u4{0u, 0u, 0u, 0u};
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            // column e of the lane's 8 x 8 block: token pairs (0,1), (2,3), (4,5), (6,7)
            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
            u4 col8;
#pragma unroll
            for (int pr = 0; pr < 4; ++pr)
                col8[pr] = __builtin_amdgcn_perm(xb[i][2 * pr + 1][e >> 1], xb[i][2 * pr][e >> 1], sel);
            if constexpr (ANY) {
                // The smallest operand first: a step of 32 rows then ends with one rounding at the size of the result.  What is not
                // finite in x is counted with the hi operand; the others, whose signs may differ, meet the largest finite number.
                const h8 fin8 = clamp_finite(as_h8(col8));
#pragma unroll
                for (int s = NS - 1; s >= 0; --s) {
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        acc[rb][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(s == 0 ? as_h8(col8) : fin8, as_h8(hl[i][rb][s]), acc[rb][e], 0, 0, 0);
                }
            } else {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    acc[rb][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(col8), as_h8(hl[i][rb][0]), acc[rb][e], 0, 0, 0);
                    acc[rb][e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(col8), as_h8(hl[i][rb][1]), acc[rb][e], 0, 0, 0);
                }
            }
        }
    };
    // t_pad and tw are multiples of 32 G: a wave's range is a whole number of groups (possibly none).  The small loads of a
    // group are requested before the x loads that are issued while the previous group is consumed, so the conversion (a
    // dependent chain of vector-ALU work and two cross-lane exchanges) never waits for x.
    if (tk_begin < tk_end) {
        issue_small(tk_begin);
#pragma unroll
        for (int i = 0; i < G; ++i) issue_x(i, tk_begin + 32 * i);
        int tk = tk_begin;
        if constexpr (ANY) {
            // One copy of the step, with the requests for the next one under a branch (4100 x 2049 -> 1001, r = 32 42.9 us, with the
            // last step apart 43.9; short batches the same).
            for (; tk < tk_end; tk += 32 * G) {
                const bool more = tk + 32 * G < tk_end;   // scalar
                convert(tk);
                if (more) issue_small(tk + 32 * G);
#pragma unroll
                for (int i = 0; i < G; ++i) {
                    consume_x(i, tk + 32 * i);
                    if (more) issue_x(i, tk + 32 * (G + i));
                }
            }
        } else {
            for (; tk + 32 * G < tk_end; tk += 32 * G) {
                convert(tk);
                issue_small(tk + 32 * G);
#pragma unroll
                for (int i = 0; i < G; ++i) {
                    consume_x(i, tk + 32 * i);
                    issue_x(i, tk + 32 * (G + i));
                }
            }
            convert(tk);
#pragma unroll
            for (int i = 0; i < G; ++i) consume_x(i, tk + 32 * i);
        }
    }

    // Accumulator e, register i of lane (li, q): rank rb*16 + li, column 8 (4q + i) + e of the block.  Each wave brings its
    // tile back to true scale; the tiles are summed in wave order; with 4 waves wave w sums register i = w of all 8
    // accumulators and so ends up with 8 consecutive columns, with 8 waves it sums register i = w mod 4 of accumulators
    // 4 (w / 4) .. 4 (w / 4) + 3: 4 consecutive columns.
    float* out = a.part + (static_cast<size_t>(blockIdx.y) * blocks + rb0) * 16 * a.dcols + static_cast<size_t>(cb) * 128;
    constexpr int NE = W == 4 ? 8 : 4;
    const int ri = wave & 3, e0 = W == 4 ? 0 : 4 * (wave >> 2);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        if (Z > 1 && rb0 + rb >= blocks) break;   // (uniform)
        if (rb > 0) __syncthreads();
        const float inv = __uint_as_float(static_cast<uint32_t>(cur_e[rb] - 13) << 23);
#pragma unroll
        for (int e = 0; e < 8; ++e) *reinterpret_cast<f4*>(&red[wave][e][lane][0]) = acc[rb][e] * inv * (ANY ? 1.f : beta[rb]);   // (one after the other: their product may vanish)
        __syncthreads();
        float sum[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            float s = red[0][e0 + e][lane][ri];
#pragma unroll
            for (int w = 1; w < W; ++w) s += red[w][e0 + e][lane][ri];
            sum[e] = s;
        }
        float* dst = out + static_cast<size_t>(rb * 16 + li) * a.dcols + 8 * (4 * q + ri) + e0;
        *reinterpret_cast<f4*>(dst) = f4{sum[0], sum[1], sum[2], sum[3]};
        if constexpr (NE == 8) *reinterpret_cast<f4*>(dst + 4) = f4{sum[4], sum[5], sum[6], sum[7]};
    }
}

// The same contraction with the tokens streamed through LDS (plain variants only).  A workgroup takes one column block and one range of
// tokens, TG tiles of 32 tokens per turn; the waves of a tile share it, each for one of the B rank blocks, so that x (or g) passes through a
// compute unit once whatever the number of rank blocks is.  The tiles come by direct loads into LDS, kTurns turns of them (the one in work among
// them): the depth costs no registers.  The sums of the TG waves of a rank block are added through LDS at the end.
// LDS of a tile: 32 rows of 256 bytes; then per rank block its 16 x 32 entries of du (or t), pieces of four tokens by rank.
// Waits: a wave's own loads of a turn are complete when at most those of the turn behind it are left (they complete in order), everybody's
// behind the barrier; the place of the turn before, which everybody has read by then, takes the next one.
// Bound: a wave's chain per tile (LDS, largest entry, conversion, 32 permutes, 16 MFMAs: about 0.5 us with two waves per SIMD) more than the
// loads (8 KB of x and 2 KB per rank block), and launch, first tile, sums and stores.  2048 x 5120 x 5120, two envelopes at r = 32: 20.2 us in a
// kernel trace, the register kernel 23.2; the whole backward call, with the finish kernel below, 44.0 (50.4), at T = 8192, r = 64 114 (136).  With two
// waves per rank block, which convert its operands twice for half of the columns each, it was a third slower, with one turn more in
// flight no faster.
constexpr int kTurns = 3;
template <int B, int TG>
__global__ __launch_bounds__(B * TG * 64) void lordba_bwd_wgrad_stream_kernel(BwdArgs a, int range) {
    constexpr int W = B * TG, NX = 8 / B, NSM = 2, PER = NX + NSM;   // waves; 1024-byte loads of a wave per turn: x, small
    constexpr int kTileBytes = 8192 + B * 2048, kSlotBytes = TG * kTileBytes;
    static_assert(W <= 16 && NX * B == 8 && PER < 64, "whole loads per wave, counted by vmcnt");
    static_assert((TG - 1) * B * 8192 <= kTurns * kSlotBytes, "the sums of the other token groups");
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, q = lane >> 4;
    if (wave == 0) clear_rank_arrivals(a, lane);
    const int rbe = a.rp >> 4, blocks = a.ell * rbe;
    const int cb = blockIdx.x, rbw = wave % B, tg = wave / B;
    const bool is_x = cb < a.nbx;
    const int d = is_x ? a.d_in : a.d_out, col0 = (is_x ? cb : cb - a.nbx) * 128;
    const _Float16* src = is_x ? a.x : a.g;
    const float* small = is_x ? a.duT : a.tT;   // du meets x, t meets g
    const int sstride = is_x ? a.du_stride : a.t_stride;
    const int64_t tk_first = static_cast<int64_t>(blockIdx.y) * range, tk_last = (static_cast<int64_t>(a.T) + 31) & ~31ll;
    const int tk_begin = static_cast<int>(tk_first < tk_last ? tk_first : tk_last);
    const int tk_end = static_cast<int>(tk_first + range < tk_last ? tk_first + range : tk_last);
    const int tiles = tk_begin < tk_end ? (tk_end - tk_begin) >> 5 : 0;

    // the lane's row of the small arrays in its loads (rank block, rank) and its own rank
    auto row_of = [&](int b, int rank) {   // (past the last block or rank: one that exists, its sums are never used)
        b = b < blocks ? b : blocks - 1;
        const int en = b / rbe, rk = (b - en * rbe) * 16 + rank;
        return en * a.r + (rk < a.r ? rk : a.r - 1);
    };
    const int my_block = rbw < blocks ? rbw : blocks - 1, my_rank = (my_block % rbe) * 16 + li;
    const float beta = my_rank < a.r ? static_cast<float>(a.s_rank[row_of(rbw, li)]) : 1.f;   // (a padded rank's sums are never used)
    const float* srow[NSM];
#pragma unroll
    for (int k = 0; k < NSM; ++k) {   // load j (two per rank block of a tile): pieces 4 (j % 2) .. of the 16 ranks of block j / 2 % B
        const int j = (wave + k * W) % (2 * B * TG);
        srow[k] = small + static_cast<size_t>(row_of((j >> 1) % B, li)) * sstride + ((j & 1) * 4 + q) * 4;
    }
    auto first_token = [&](int i, int tile) {   // of tile `tile` of turn i (behind the last tile: it again, not used)
        const int at = i * TG + tile;
        return tk_begin + 32 * (at < tiles ? at : tiles - 1);
    };
    auto issue = [&](int i) {
        const uint32_t slot = static_cast<uint32_t>(i % kTurns) * kSlotBytes;
#pragma unroll
        for (int k = 0; k < NX; ++k) {   // four rows of a tile
            const int j = wave + k * W, r = 4 * (j & 7) + q;
            int row = first_token(i, j >> 3) + r, col = col0 + li * 8;
            row = row < a.T ? row : a.T - 1;   // rows past T meet du = t = 0
            col = col < d ? col : d - 8;       // past the end: a valid piece is re-read, its sums are never used
            const _Float16* p = src + static_cast<size_t>(row) * d + col;
            load16_to_lds<true>(slot + (j >> 3) * kTileBytes + (j & 7) * 1024u, p);
        }
#pragma unroll
        for (int k = 0; k < NSM; ++k) {
            const int j = (wave + k * W) % (2 * B * TG), tile = j / (2 * B);
            load16_to_lds<false>(slot + tile * kTileBytes + 8192u + (j % (2 * B)) * 1024u, srow[k] + first_token(i, tile));
        }
    };
    // (the products with the lo operands have sums of their own: one rounding per tile at the size of the result instead of two.  Error of the
    // latent gradients against 64 bits, T = 2048, 4096^2, r = 64: 2.15e-7, in one sum 2.4e-7, in the kernel above 2.2e-7)
    f4 acc[8], acc_lo[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = acc_lo[e] = f4{0.f, 0.f, 0.f, 0.f};
    int cur_e = 14;   // (the power-of-two scaling per rank of the kernel above; beta comes in at the end)
    const bool silent = __builtin_amdgcn_ballot_w64(beta == 0.f) != 0ull;   // a rank without scale: it adds nothing, whatever its entries are
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (beta: from here on the loads are counted)
    const int turns = (tiles + TG - 1) / TG;
#pragma unroll 1
    for (int i = 0; i < kTurns - 1 && i < turns; ++i) issue(i);
#pragma unroll 1
    for (int i = 0; i < turns; ++i) {
        if (i + 1 < turns) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(PER) : "memory");   // (one turn is behind this one: the next is issued below)
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (i + kTurns - 1 < turns) issue(i + kTurns - 1);
        if (i * TG + tg >= tiles) continue;   // (scalar)
        const unsigned char* slot = smem + (i % kTurns) * kSlotBytes + tg * kTileBytes;
        float v[8];
        {
            const unsigned char* sp = slot + 8192 + rbw * 2048 + (2 * q * 16 + li) * 16;
            const u4 s0 = load16(sp), s1 = load16(sp + 256);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(e < 4 ? s0[e & 3] : s1[e & 3]);
        }
        const int tk = first_token(i, tg) + 8 * q;
        if (silent || first_token(i, tg) + 32 > a.T) {   // scalar: the last rows (entries past T are undefined)
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = beta != 0.f && tk + e < a.T ? v[e] : 0.f;
        }
        if (const float f = follow_largest(v, cur_e); __builtin_amdgcn_ballot_w64(f != 1.f) != 0ull) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                acc[e] *= f;
                acc_lo[e] *= f;
            }
        }
        u4 hi, lo;
        split_scaled(v, __uint_as_float(static_cast<uint32_t>(267 - cur_e) << 23), hi, lo);
        u4 xr[8];   // token rows 8 q + e of the lane's 8 columns
#pragma unroll
        for (int e = 0; e < 8; ++e) xr[e] = load16(slot + (8 * q + e) * 256 + li * 16);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
            u4 col8;
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) col8[pr] = __builtin_amdgcn_perm(xr[2 * pr + 1][e >> 1], xr[2 * pr][e >> 1], sel);
            acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(col8), as_h8(hi), acc[e], 0, 0, 0);
            acc_lo[e] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(col8), as_h8(lo), acc_lo[e], 0, 0, 0);
        }
    }
    // Accumulator e, register i of lane (li, q): rank li, column 8 (4 q + i) + e: 32 consecutive columns per lane
    const float back = __uint_as_float(static_cast<uint32_t>(cur_e - 13) << 23);
    float out[32];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int e = 0; e < 8; ++e) out[i * 8 + e] = (acc[e][i] + acc_lo[e][i]) * back * beta;   // (one after the other: their product may vanish)
    }
    if constexpr (TG > 1) {   // the token groups' sums, in their order
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();
        f4* red = reinterpret_cast<f4*>(smem);
        if (tg > 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) red[(((tg - 1) * B + rbw) * 8 + i) * 64 + lane] = f4{out[4 * i], out[4 * i + 1], out[4 * i + 2], out[4 * i + 3]};
        }
        __syncthreads();
        if (tg > 0) return;
#pragma unroll
        for (int t = 1; t < TG; ++t) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const f4 o = red[(((t - 1) * B + rbw) * 8 + i) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) out[4 * i + e] += o[e];
            }
        }
    }
    if (rbw >= blocks) return;   // (a rank block too many)
    float* dst = a.part + ((static_cast<size_t>(blockIdx.y) * blocks + rbw) * 16 + li) * a.dcols + static_cast<size_t>(cb) * 128 + 32 * q;
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<f4*>(dst + 4 * i) = f4{out[4 * i], out[4 * i + 1], out[4 * i + 2], out[4 * i + 3]};
}

// ---------------------------------------------------------------------------------------- finish kernel ----
// kappa (1 - tanh^2(z)) = 4 kappa e / (1 + e)^2 with e = exp(-2 |z|): no cancellation at large |z|.
__device__ __forceinline__ float smooth_sign_factor(float latent, float kappa) {
    const float e = expf(-2.f * fabsf(kappa * latent));
    const float s = 1.f + e;
    return 4.f * kappa * e / (s * s);
}

// sum_t du[t] t[t] over tokens begin .. end - 1 of row k by the threads of a workgroup: this thread's share.
template <int NT>
__device__ __forceinline__ float token_sum(const BwdArgs& a, int k, int64_t begin, int64_t end) {
    const float* du = a.duT + static_cast<size_t>(k) * a.du_stride;
    const float* t = a.tT + static_cast<size_t>(k) * a.t_stride;
    constexpr int U = 4;   // pieces of four tokens in flight
    auto piece = [&](const float* p, int tok) { return drop_words(load16_word(p + row_piece(tok, a.T, k)), tok - row_piece(tok, a.T, k)); };
    float acc[U][4];
#pragma unroll
    for (int j = 0; j < U; ++j) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = 0.f;
    }
    for (int64_t i = begin + 4 * threadIdx.x; i < end; i += 4 * U * NT) {
        u4 dv[U], tv[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int tok = static_cast<int>(i + 4 * j * NT < end ? i + 4 * j * NT : i);
            dv[j] = piece(du, tok);
            tv[j] = piece(t, tok);
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
#pragma unroll
            for (int e = 0; e < 4; ++e)   // select: entries past T are undefined
                acc[j][e] += i + 4 * j * NT + e < end ? __uint_as_float(dv[j][e]) * __uint_as_float(tv[j][e]) : 0.f;
        }
    }
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < U; ++j) s += (acc[j][0] + acc[j][1]) + (acc[j][2] + acc[j][3]);
    return s;
}
// Sum over the threads of a workgroup, in the first one (fixed order: wave, waves).
template <int NT>
__device__ __forceinline__ float workgroup_sum(float s, float* red) {
#pragma unroll
    for (int step = 32; step >= 1; step >>= 1) s += __shfl_xor(s, step, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    float tot = 0.f;
    if (threadIdx.x == 0)
        for (int w = 0; w < NT / 64; ++w) tot += red[w];
    return tot;
}

// d_beta_k = sum_t du[t, k] t[t, k], workgroup wg of rank_parts for each of the ranks of all envelopes.  (By the wgrad kernel's workgroups of one
// column block it was up to 5 us behind their other work, up to 20 on narrow batches.)  The last one of a rank to arrive adds the parts up, in
// their order, so the order of the sum is fixed: thread, wave, waves, parts.  One workgroup per rank, whatever T is, keeps the launch waiting on
// long batches: see rank_parts.
template <int NT>
__device__ __forceinline__ void rank_scale_gradient(const BwdArgs& a, int wg, float* red) {
    const int parts = a.rank_parts, k = parts == 1 ? wg : wg / parts, part = wg - k * parts;
    const int64_t begin = static_cast<int64_t>(part) * a.rank_tokens, end = begin + a.rank_tokens < a.T ? begin + a.rank_tokens : a.T;
    float tot = workgroup_sum<NT>(token_sum<NT>(a, k, begin, end), red);
    if (parts > 1) {
        uint32_t* last = reinterpret_cast<uint32_t*>(red) + NT / 64;
        float* sums = a.rank_sums + a.ell * a.rp + k;   // (the arrivals are in front of them)
        if (threadIdx.x == 0) {
            __hip_atomic_store(sums + part * a.ell * a.rp, tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            *last = __hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(a.rank_sums) + k, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == static_cast<uint32_t>(parts);
        }
        __syncthreads();
        if (*last == 0u) return;
        const int mine = static_cast<int>(threadIdx.x) < parts ? threadIdx.x : 0;
        const float v = __hip_atomic_load(sums + mine * a.ell * a.rp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        tot = workgroup_sum<NT>(static_cast<int>(threadIdx.x) < parts ? v : 0.f, red);
    }
    if (threadIdx.x == 0) a.d_s_rank[k] = tot;
}
template <int RK>
constexpr int kFinishThreads = RK < 32 ? 256 : 8 * RK;
template <int L>
constexpr int kFinishShares = L == 1 ? 8 : 4;   // token ranges' shares that a thread has in flight
// Widths that are multiples of 32.  A workgroup takes NG groups of 32 columns of d_in (Q, d_s_in, d_latentA) or of d_out (P, d_s_out,
// d_latentB); a thread takes four columns and one rank (RK >= r of them), with all envelopes' shares, so that everything it needs is requested at
// once in 16-byte pieces (up to eight token ranges with one envelope, four with more).  The workgroups in front of these take d_s_rank.  Bound: one
// trip to memory behind the launch.  2048 x 5120 x 5120, two envelopes at r = 32 5.2 us in a kernel trace, with one column per thread, shares eight
// at a time per envelope and latentB through LDS first 8.5; 4096^2, r = 16 4.5 (4.5).
// Where there are more token ranges than that a workgroup takes one group instead, KS threads per entry with every KS-th range each: more
// ranges mean fewer column blocks (512 workgroups in all), few workgroups of several groups, and a trip per eight (or four) ranges.  us, several
// groups in brackets: this kernel at 8192 x 1024 x 1024, r = 4, 32 ranges 3.8 (5.3), 1048576 x 64 x 64, r = 1, 256 ranges 6.8 (20.1); the backward call there
// 30.1 (32.8), 880 (890), at 4096 x 256 x 256, r = 16 18.8 (21.8), two envelopes at r = 16 8192 x 256 x 256 33.2 (35.8), 1000 x 2048 x 2048 21.8 (22.7).
template <int RK, int L, int KS>
__global__ __launch_bounds__(kFinishThreads<RK>) void lordba_bwd_finish_kernel(BwdArgs a) {
    constexpr int NT = kFinishThreads<RK>, NG = NT / (8 * RK * KS), SP = kFinishShares<L>;
    __shared__ __align__(16) float sh[NG][L][RK][32];
    __shared__ float lat[NG][32 * RK];
    __shared__ __align__(16) float others[KS > 1 ? KS - 1 : 1][L][RK][32];
    static_assert(NG * KS * 8 * RK == NT && NG * 32 * RK > NT / 64, "whole groups; room for a workgroup's sums of d_s_rank");
    const int tid = threadIdx.x, r = a.r, rows = L * a.rp, in_front = L * r * a.rank_parts;
    if (static_cast<int>(blockIdx.x) < in_front) {
        rank_scale_gradient<NT>(a, blockIdx.x, &lat[0][0]);
        return;
    }
    const int gx = a.d_in >> 5, gg = a.d_out >> 5;
    const int part = __builtin_amdgcn_readfirstlane(tid / (8 * RK)), ng = KS > 1 ? 0 : part, ks = KS > 1 ? part : 0;   // group, or part of its shares
    const int k = (tid >> 3) & (RK - 1), c = (tid & 7) * 4;   // rank, first of the four columns
    const int g0 = (static_cast<int>(blockIdx.x) - in_front) * NG + ng;
    const bool live = g0 < gx + gg && k < r;
    const int gc = g0 < gx + gg ? g0 : gx + gg - 1, kc = k < r ? k : r - 1;   // (a group and a rank that exist)
    const bool is_x = gc < gx;
    const int grp = is_x ? gc : gc - gx, d = is_x ? a.d_in : a.d_out, col = grp * 32 + c;
    const bool with_lat = a.d_latA != nullptr;   // (null: the carriers are frozen, only the scale gradients are wanted)
    const float* plane = a.part + static_cast<size_t>(kc) * a.dcols + (is_x ? col : a.nbx * 128 + col);
    const size_t plane_stride = static_cast<size_t>(rows) * a.dcols, env_stride = static_cast<size_t>(a.rp) * a.dcols;
    f4 sum[L];
    u4 v[L][SP];
    auto request = [&](int sp0) {
#pragma unroll
        for (int en = 0; en < L; ++en) {
#pragma unroll
            for (int j = 0; j < SP; ++j) {
                const int at = (sp0 + j) * KS + ks, sp = at < a.splits ? at : a.splits - 1;
                v[en][j] = load16(plane + sp * plane_stride + en * env_stride);
            }
        }
    };
    request(0);
    const uint32_t word = (is_x ? a.pA : a.pBt)[kc * (d >> 5) + grp] >> c;
    uint2 scale[L];
#pragma unroll
    for (int en = 0; en < L; ++en)
        scale[en] = *reinterpret_cast<const uint2*>((is_x ? a.s_in : a.s_out) + static_cast<size_t>(en) * d + col);
    float latent[4] = {0.f, 0.f, 0.f, 0.f};
    if (with_lat && ks == 0) {
        if (is_x) {   // (the same in all lanes of a wave: a group has at least one of its own)
            const u4 w = *reinterpret_cast<const u4_word*>(a.latA + static_cast<size_t>(kc) * d + col);
#pragma unroll
            for (int e = 0; e < 4; ++e) latent[e] = __uint_as_float(w[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) latent[e] = a.latB[static_cast<size_t>(col + e) * r + kc];
        }
    }
#pragma unroll
    for (int en = 0; en < L; ++en) sum[en] = f4{0.f, 0.f, 0.f, 0.f};
    for (int sp0 = 0;; sp0 += SP) {
#pragma unroll
        for (int en = 0; en < L; ++en) {
#pragma unroll
            for (int j = 0; j < SP; ++j) {
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[en][e] += (sp0 + j) * KS + ks < a.splits ? __uint_as_float(v[en][j][e]) : 0.f;
            }
        }
        if ((sp0 + SP) * KS >= a.splits) break;
        request(sp0 + SP);
    }
    if constexpr (KS > 1) {   // the parts' sums, in their order
        if (ks > 0) {
#pragma unroll
            for (int en = 0; en < L; ++en) *reinterpret_cast<f4*>(&others[ks - 1][en][k][c]) = sum[en];
        }
        __syncthreads();
        if (ks == 0) {
#pragma unroll
            for (int o = 0; o < KS - 1; ++o) {
#pragma unroll
                for (int en = 0; en < L; ++en) sum[en] += *reinterpret_cast<const f4*>(&others[o][en][k][c]);
            }
        }
    }
    float weighted[4] = {0.f, 0.f, 0.f, 0.f};   // sum over the envelopes of scale_e * (Q_e or P_e)[k, col]: dL/dS[k, col]
#pragma unroll
    for (int en = 0; en < L; ++en) {
        f4 ds;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float sc = static_cast<float>(as_h2(e < 2 ? scale[en].x : scale[en].y)[e & 1]);
            ds[e] = live ? flip(sum[en][e], (word >> e) & 1u) : 0.f;
            weighted[e] = L == 1 ? sc * sum[en][e] : fmaf(sc, sum[en][e], weighted[e]);
        }
        if (ks == 0) *reinterpret_cast<f4*>(&sh[ng][en][k][c]) = ds;
    }
    if (with_lat && live && ks == 0) {
        float val[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) val[e] = weighted[e] * smooth_sign_factor(latent[e], a.kappa);
        if (is_x) {
            u4_word* dst = reinterpret_cast<u4_word*>(a.d_latA + static_cast<size_t>(k) * d + col);
            u4 w;
            if (a.accumulate) w = *dst;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = __float_as_uint(a.accumulate ? __uint_as_float(w[e]) + val[e] : val[e]);
            *dst = w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) lat[ng][(c + e) * r + k] = val[e];   // (the group's 32 r entries of d_latentB, in their order)
        }
    }
    __syncthreads();
    constexpr int GT = 8 * RK * KS;
    const int gt = tid & (GT - 1);   // thread of the group
    if (g0 >= gx + gg) return;
    if (with_lat && !is_x) {
        float* dst = a.d_latB + static_cast<size_t>(grp) * 32 * r;
        for (int e = gt; e < 32 * r; e += GT) dst[e] = a.accumulate ? dst[e] + lat[ng][e] : lat[ng][e];
    }
    for (int o = gt; o < 32 * L; o += GT) {   // the sums over the ranks, in their order
        const int en = o >> 5, cc = o & 31;
        float tot[4] = {0.f, 0.f, 0.f, 0.f};   // (four sums of a quarter of the ranks each: a chain over 64 would round more often)
#pragma unroll 4
        for (int j = 0; j < RK; j += 4) {
#pragma unroll
            for (int m = 0; m < 4; ++m) tot[m] += sh[ng][en][j + m][cc];
        }
        (is_x ? a.d_s_in : a.d_s_out)[static_cast<size_t>(en) * d + grp * 32 + cc] = (tot[0] + tot[1]) + (tot[2] + tot[3]);
    }
}

// Any widths: one workgroup per group of 32 columns of d_in (Q, d_s_in, d_latentA) or of d_out (P, d_s_out, d_latentB), behind those for
// d_s_rank.  Thread (c, kq) takes column c of the group and ranks kq, kq + KQ, ...; every sum has a fixed order.  KQ is the
// padded rank up to 32: a thread then has one or two dependent rounds of requests instead of r / 8.
template <int KQ>
__global__ __launch_bounds__(32 * KQ) void lordba_bwd_finish_any_kernel(BwdArgs a) {
    constexpr int NT = 32 * KQ;
    __shared__ float sh[LORDBA_MAX_ENVELOPES][NT];
    __shared__ float lat[32 * LORDBA_MAX_RANK];
    const int gx = (a.d_in + 31) >> 5;
    const int tid = threadIdx.x;
    const int r = a.r, ell = a.ell, rows = ell * a.rp;   // rows of one token range's plane of partial sums: all envelopes' rank blocks
    const int in_front = ell * r * a.rank_parts;
    if (static_cast<int>(blockIdx.x) < in_front) {
        rank_scale_gradient<NT>(a, blockIdx.x, sh[0]);
        return;
    }
    const int wg = static_cast<int>(blockIdx.x) - in_front;
    const bool is_x = wg < gx;
    const int grp = is_x ? wg : wg - gx;
    const int d = is_x ? a.d_in : a.d_out;
    const int c = tid & 31, kq = tid >> 5;
    const bool live = grp * 32 + c < d;   // (the last group may have fewer than 32 columns)
    const int col = live ? grp * 32 + c : d - 1;
    const float* plane = a.part + (is_x ? col : a.nbx * 128 + col);
    const uint32_t* pk = is_x ? a.pA : a.pBt;   // both [r, d]: the group's 32 bits of rank k are one word
    float scale[LORDBA_MAX_ENVELOPES], dscale[LORDBA_MAX_ENVELOPES];
#pragma unroll
    for (int en = 0; en < LORDBA_MAX_ENVELOPES; ++en) {
        const int ec = en < ell ? en : 0;
        scale[en] = static_cast<float>(is_x ? a.s_in[static_cast<size_t>(ec) * d + col] : a.s_out[static_cast<size_t>(ec) * d + col]);
        dscale[en] = 0.f;
    }
    const int lat_n = (d - grp * 32 < 32 ? d - grp * 32 : 32) * r;
    if (!is_x && a.d_latB != nullptr) {  // latentB [d_out, r]: the group's 32 rows are 32 r contiguous floats; through LDS for coalesced accesses
        for (int e = tid; e < lat_n; e += NT) lat[e] = a.latB[static_cast<size_t>(grp) * 32 * r + e];
        __syncthreads();
    }
    const bool with_lat = a.d_latA != nullptr;   // (null: the carriers are frozen, only the scale gradients are wanted)
    const bool lat_x = with_lat && is_x, add_x = lat_x && a.accumulate;
    for (int k = kq; k < r; k += KQ) {
        // Everything this rank needs is requested before anything is used: the shares of the token ranges (eight at a
        // time, from a clamped index), the carrier word, the latent and, when accumulating, the gradient so far.  The
        // last two come from a harmless address when they are not wanted, so that no request hides behind a branch.
        const size_t n = static_cast<size_t>(k) * d + col;
        const uint32_t word = pk[n >> 5];
        const float latent = *(lat_x ? a.latA + n : plane);
        const float so_far = *(add_x ? a.d_latA + n : plane);
        const uint32_t bit = (word >> static_cast<int>(n & 31)) & 1u;
        float weighted = 0.f;   // sum over the envelopes of scale_e * (Q_e or P_e)[k, col]: dL/dS[k, col]
#pragma unroll
        for (int en = 0; en < LORDBA_MAX_ENVELOPES; ++en) {
            if (en < ell) {
                float s = 0.f;
                for (int sp0 = 0; sp0 < a.splits; sp0 += 8) {
                    float v[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int sp = sp0 + j < a.splits ? sp0 + j : a.splits - 1;
                        v[j] = plane[(static_cast<size_t>(sp) * rows + en * a.rp + k) * a.dcols];
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) s += (sp0 + j < a.splits) ? v[j] : 0.f;
                }
                dscale[en] += flip(s, bit);
                weighted = ell == 1 ? scale[0] * s : fmaf(scale[en], s, weighted);
            }
        }
        if (lat_x) {
            const float val = weighted * smooth_sign_factor(latent, a.kappa);
            if (live) a.d_latA[n] = add_x ? so_far + val : val;
        } else if (with_lat && live) {
            lat[c * r + k] = weighted * smooth_sign_factor(lat[c * r + k], a.kappa);
        }
    }
#pragma unroll
    for (int en = 0; en < LORDBA_MAX_ENVELOPES; ++en) sh[en][tid] = dscale[en];
    __syncthreads();
    if (!is_x && a.d_latB != nullptr)
        for (int e = tid; e < lat_n; e += NT) {
            float* dst = a.d_latB + static_cast<size_t>(grp) * 32 * r + e;
            *dst = a.accumulate ? *dst + lat[e] : lat[e];
        }
    if (kq < ell && live) {   // wave pair kq sums envelope kq's partial sums of every column
        float tot = 0.f;
#pragma unroll
        for (int j = 0; j < KQ; ++j) tot += sh[kq][j * 32 + c];
        (is_x ? a.d_s_in : a.d_s_out)[static_cast<size_t>(kq) * d + col] = tot;
    }
}

// --------------------------------------------------------------------------------------- general kernel ----
// Q, P and everything that follows from them for widths below 8 columns, for a kept t whose rows end before the padded token
// count and for the fewest rows (backward_impl), on the vector ALU: one thread per column of x (Q[:, i], then d_s_in[i] and
// d_latentA[:, i]) or of g (P[:, j], d_s_out[j], d_latentB[j, :]) walks all token rows with its r sums in registers; r more threads take d_s_rank.  No partial sums, fixed order.  Slow (a column's T x r
// multiply-adds in one thread) but it takes every shape.
template <int RP>
__global__ __launch_bounds__(256) void lordba_bwd_general_kernel(BwdArgs a) {
    __shared__ float beta_s[RP];
    const int r = a.r, tid = threadIdx.x;
    if (tid < RP) beta_s[tid] = tid < r ? static_cast<float>(a.s_rank[tid]) : 0.f;
    __syncthreads();
    const int64_t c = static_cast<int64_t>(blockIdx.x) * 256 + tid;
    const int64_t ncols = static_cast<int64_t>(a.d_in) + a.d_out;
    if (c >= ncols + r) return;
    if (c >= ncols) {  // d_beta_k = sum_t du[t, k] t[t, k]
        const int k = static_cast<int>(c - ncols);
        const float* dup = a.duT + static_cast<size_t>(k) * a.du_stride;
        const float* tp = a.tT + static_cast<size_t>(k) * a.t_stride;
        float s = 0.f;
        for (int t = 0; t < a.T; ++t) s = fmaf(dup[t], tp[t], s);
        a.d_s_rank[k] = s;
        return;
    }
    const bool is_x = c < a.d_in;
    const int col = static_cast<int>(is_x ? c : c - a.d_in);
    const int d = is_x ? a.d_in : a.d_out;
    const _Float16* src = (is_x ? a.x : a.g) + col;
    const float* small = is_x ? a.duT : a.tT;   // dt = beta du meets x, u = beta t meets g
    const int sstride = is_x ? a.du_stride : a.t_stride;
    float acc[RP];
#pragma unroll
    for (int k = 0; k < RP; ++k) acc[k] = 0.f;
    for (int t = 0; t < a.T; ++t) {
        const float v = static_cast<float>(src[static_cast<size_t>(t) * d]);
#pragma unroll
        for (int k = 0; k < RP; ++k)
            if (k < r) acc[k] = fmaf(small[static_cast<size_t>(k) * sstride + t] * beta_s[k], v, acc[k]);
    }
    const uint32_t* pk = is_x ? a.pA : a.pBt;   // both [r, d] bit streams
    const float scale = static_cast<float>(is_x ? a.s_in[col] : a.s_out[col]);
    const bool with_lat = a.d_latA != nullptr;
    float dscale = 0.f;
#pragma unroll
    for (int k = 0; k < RP; ++k) {
        if (k < r) {
            const int64_t n = static_cast<int64_t>(k) * d + col;
            dscale += flip(acc[k], (pk[n >> 5] >> (n & 31)) & 1u);
            if (with_lat) {
                const size_t at = is_x ? static_cast<size_t>(n) : static_cast<size_t>(col) * r + k;   // latentA [r, d_in], latentB [d_out, r]
                const float* lat = is_x ? a.latA : a.latB;
                float* out = is_x ? a.d_latA : a.d_latB;
                const float val = scale * acc[k] * smooth_sign_factor(lat[at], a.kappa);
                out[at] = a.accumulate ? out[at] + val : val;
            }
        }
    }
    (is_x ? a.d_s_in : a.d_s_out)[col] = dscale;
}

template <int RP>
lordba_status launch_general(const BwdArgs& a, hipStream_t st) {
    const int64_t n = static_cast<int64_t>(a.d_in) + a.d_out + a.r;
    hipLaunchKernelGGL((lordba_bwd_general_kernel<RP>), dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? LORDBA_OK : LORDBA_ERR_LAUNCH;
}

// ------------------------------------------------------------------------------------------ host side ----
bool aligned_to(const void* p, size_t n) { return (reinterpret_cast<uintptr_t>(p) & (n - 1)) == 0; }

template <int KQ>
void launch_finish_any(const BwdArgs& a, hipStream_t st) {
    const dim3 groups(a.ell * a.r * a.rank_parts + (a.d_in + 31) / 32 + (a.d_out + 31) / 32);
    hipLaunchKernelGGL((lordba_bwd_finish_any_kernel<KQ>), groups, dim3(32 * KQ), 0, st, a);
}
template <int RK, int L, int KS>
void launch_finish_parts(const BwdArgs& a, hipStream_t st) {
    constexpr int NT = kFinishThreads<RK>, NG = NT / (8 * RK * KS);
    const unsigned groups = static_cast<unsigned>(a.d_in / 32 + a.d_out / 32);
    hipLaunchKernelGGL((lordba_bwd_finish_kernel<RK, L, KS>), dim3(L * a.r * a.rank_parts + (groups + NG - 1) / NG), dim3(NT), 0, st, a);
}
template <int RK, int L>
void launch_finish(const BwdArgs& a, hipStream_t st) {
    constexpr int KS = kFinishThreads<RK> / (8 * RK);
    if constexpr (KS > 1)
        if (a.splits > kFinishShares<L>) return launch_finish_parts<RK, L, KS>(a, st);
    launch_finish_parts<RK, L, 1>(a, st);
}
template <int L>
void launch_finish_rank(const BwdArgs& a, hipStream_t st) {
    // (four rank blocks at most in all: two envelopes have ranks up to 32, three and four up to 16)
    if (a.r <= 8) return launch_finish<8, L>(a, st);
    if constexpr (L <= 2)
        if (a.r > 32 && L == 1) return launch_finish<64, 1>(a, st);
    if constexpr (L <= 2)
        if (a.r > 16) return launch_finish<32, L>(a, st);
    launch_finish<16, L>(a, st);
}

template <int RB, int W, int Z, bool ANY>
lordba_status launch_wgrad(const BwdArgs& a, hipStream_t st) {
    const int nb = a.nbx + a.nbg;
    const dim3 grid(Z > 1 ? (nb + 7) / 8 * 8 * Z : nb, a.splits);
    hipLaunchKernelGGL((lordba_bwd_wgrad_kernel<RB, kWgradGroup, W, Z, ANY>), grid, dim3(W * 64), 0, st, a);
    return LORDBA_OK;
}
template <int B, int TG>
lordba_status launch_stream(const BwdArgs& a, int64_t range, hipStream_t st) {
    constexpr size_t lds = kTurns * TG * (8192 + B * 2048);
    auto kern = lordba_bwd_wgrad_stream_kernel<B, TG>;
    {   // more than 64 KiB of LDS per workgroup, asked for once per device
        static std::mutex mu;
        static bool granted[64] = {false};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return LORDBA_ERR_NO_DEVICE;
        std::lock_guard<std::mutex> g(mu);
        if (!granted[dev]) {
            if (hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)) != hipSuccess) {
                (void)hipGetLastError();
                return LORDBA_ERR_LAUNCH;
            }
            granted[dev] = true;
        }
    }
    hipLaunchKernelGGL(kern, dim3(a.nbx + a.nbg, a.splits), dim3(B * TG * 64), lds, st, a, static_cast<int>(range));
    return LORDBA_OK;
}

lordba_status launch_all(const BwdArgs& args, hipStream_t st) {
    BwdArgs a = args;
    const bool short_batch = a.T < kShortBatch;
    const int blocks = a.ell * (a.rp / 16);   // rank blocks of all envelopes together
    // From two rank blocks on the kernel that streams the tokens through LDS, where there is enough to stream: it starts later (tiles have to be in
    // LDS, its sums go through it at the end) and gains with every tile, of which a compute unit gets T (column blocks) / 8192.  Below, the kernel
    // that holds the tokens in registers, with a workgroup per block (or two) on short batches (Z), which read x (or g) again out of
    // the L2 they share.  us of the whole backward call, that kernel in brackets: 4096 -> 4096, T = 2000, r = 32 28.6 (30.0); 5120 -> 11008, r = 32,
    // T = 600 31.3 (31.0), 1100 39.8 (40.8), 3500 69.8 (80.9); r = 48 36.7 (37.6), 45.2 (48.0), 86.1 (101.9); r = 64 41.8 (41.4), 51.0 (52.4), 97.2 (106);
    // 1536 -> 1536, T = 1100, r = 48 23.1 (22.2), T = 2000 24.3 (25.0); T = 8192, 5120^2, r = 64 114 (136), two envelopes at r = 16 97.0 (99.5).
    // One block gains nothing (2048 x 4096^2, r = 16 25.6 (24.3), T = 8192, 13824 -> 5120 174 (169)): nothing is shared.
    const int64_t tiles = static_cast<int64_t>(a.T) * (a.nbx + a.nbg);
    const bool enough = !a.any && ((blocks == 2 && (!short_batch || tiles >= 72 * 1024)) || (blocks >= 3 && tiles >= 48 * 1024));
    // One workgroup fits a compute unit: as few token ranges as leave the last round of 256 workgroups nearly full (at least 0.9 of the
    // best that the plan, which has the room for the sums, allows), in pieces of 64 rows.  5614 x 10496 -> 6016, three envelopes at
    // r = 4, 129 column blocks: one range 170 us, three 153.
    auto filled = [&](int splits) {
        const int64_t n = static_cast<int64_t>(a.nbx + a.nbg) * splits;
        return static_cast<double>(n) / static_cast<double>((n + 255) / 256 * 256);
    };
    double best = 0.0;
    for (int k = 1; k <= a.splits; ++k) best = filled(k) > best ? filled(k) : best;
    // Not three rank blocks where that is little more than half of the chip (129 to 161 column blocks below 4096 rows, one range): a quarter of the
    // waves has nothing to do as it is, and single blocks over workgroups fill it (three envelopes at r = 4, the streamed kernel in brackets: 129
    // column blocks, T = 400 35.4 (38.5), T = 1200 62.2 (65.8), 136, T = 2000 79.6 (83.0), 154, T = 800 52.4 (53.3), but 170 59.3 (56.5)).
    const bool stream = enough && !(blocks == 3 && best < 0.63);
    int64_t range = static_cast<int64_t>(a.tw) * a.waves;   // token rows of a workgroup
    if (stream) {
        int splits = 1;
        while (splits < a.splits && filled(splits) < 0.9 * best) ++splits;
        range = ((a.T + splits - 1) / splits + 63) / 64 * 64;
        a.splits = static_cast<int>((a.T + range - 1) / range);
    }
    lordba_status s;
    if (stream) s = blocks == 2 ? launch_stream<2, 4>(a, range, st) : launch_stream<4, 2>(a, range, st);
    else if (blocks == 1 && a.waves == 2 * kWgradWaves) s = a.any ? launch_wgrad<1, 2 * kWgradWaves, 1, true>(a, st) : launch_wgrad<1, 2 * kWgradWaves, 1, false>(a, st);
    else if (blocks == 1) s = a.any ? launch_wgrad<1, kWgradWaves, 1, true>(a, st) : launch_wgrad<1, kWgradWaves, 1, false>(a, st);
    else if (!a.any) s = blocks == 2 ? launch_wgrad<1, kWgradWaves, 2, false>(a, st) : blocks == 3 && short_batch ? launch_wgrad<1, kWgradWaves, 3, false>(a, st) : launch_wgrad<2, kWgradWaves, 2, false>(a, st);
    // (A workgroup that held three or four blocks left one wave per SIMD, 462 registers, with nothing to overlap its conversions, products
    // and requests with; short batches gain from single blocks too, but not from four of them: r = 64, T = 2048 46.0 against 43.5 us.)
    else if (blocks == 2) s = short_batch ? launch_wgrad<1, kWgradWaves, 2, true>(a, st) : launch_wgrad<2, kWgradWaves, 1, true>(a, st);
    else if (blocks == 3 && short_batch) s = launch_wgrad<1, kWgradWaves, 3, true>(a, st);
    else s = launch_wgrad<2, kWgradWaves, 2, true>(a, st);
    if (s != LORDBA_OK) return s;
    if (hipGetLastError() != hipSuccess) return LORDBA_ERR_LAUNCH;
    if (a.any) {
        if (a.r <= 8) launch_finish_any<8>(a, st);
        else if (a.r <= 16) launch_finish_any<16>(a, st);
        else launch_finish_any<32>(a, st);
    } else {
        if (a.ell == 1) launch_finish_rank<1>(a, st);
        else if (a.ell == 2) launch_finish_rank<2>(a, st);
        else if (a.ell == 3) launch_finish_rank<3>(a, st);
        else launch_finish_rank<4>(a, st);
    }
    return hipGetLastError() == hipSuccess ? LORDBA_OK : LORDBA_ERR_LAUNCH;
}

bool supported(int64_t T, int64_t d_in, int64_t d_out, int64_t r) {
    return T >= 0 && d_in >= 1 && d_out >= 1 && r >= 1 && r <= LORDBA_MAX_RANK && T <= INT32_MAX - 128 && d_in <= (1 << 24) &&
           d_out <= (1 << 24);
}
// The matrix-core wgrad and the finish kernel read whole 128-column blocks and 32-column words.
bool fast_shape(int64_t d_in, int64_t d_out) { return d_in % 32 == 0 && d_out % 32 == 0; }

}  // namespace

extern "C" size_t lordba_backward_workspace_bytes(int64_t T, int64_t d_in, int64_t d_out, int64_t r) {
    if (!supported(T, d_in, d_out, r)) return 0;
    return make_plan(T, d_in, d_out, r).words * 4;
}

extern "C" size_t lordba_backward_multi_workspace_bytes(int64_t T, int64_t d_in, int64_t d_out, int64_t r, int64_t ell) {
    if (!supported(T, d_in, d_out, r) || ell < 1 || ell > LORDBA_MAX_ENVELOPES) return 0;
    const bool one_pass = ell > 1 && fast_shape(d_in, d_out) && ell * ((r + 15) / 16) <= 4;
    return make_plan(T, d_in, d_out, r, one_pass ? ell : 1).words * 4;
}

namespace {

// Shared by the entry points.  ell envelopes: s_in, s_rank, s_out and their gradients have ell rows; everything is additive
// over the envelopes (DeltaW is their sum and g is fixed), so envelope e is one pass of the one-envelope machinery with its
// own scales: its own scale gradients, and latent gradients added to those of the envelopes before it.
lordba_status backward_impl(const void* x, const void* g,
                            const uint32_t* packedA, const uint32_t* packedAt, const uint32_t* packedBt,
                            const void* s_in, const void* s_rank, const void* s_out,
                            const float* latentA, const float* latentB, float kappa,
                            const float* t_saved, int64_t t_stride,
                            const void* dx_base, void* dx,
                            float* d_s_in, float* d_s_rank, float* d_s_out,
                            float* d_latentA, float* d_latentB,
                            void* workspace, size_t workspace_bytes,
                            int64_t T, int64_t d_in, int64_t d_out, int64_t r, int64_t ell, void* stream) {
    if (!supported(T, d_in, d_out, r) || ell < 1 || ell > LORDBA_MAX_ENVELOPES) return LORDBA_ERR_DIM;
    if (!packedA || !packedAt || !packedBt || !s_in || !s_rank || !s_out || !d_s_in || !d_s_rank || !d_s_out || !workspace)
        return LORDBA_ERR_NULL;
    // frozen carriers (only the scales are trained): no latents, no latent gradients
    const bool with_latents = d_latentA != nullptr || d_latentB != nullptr;
    if (with_latents && (!latentA || !latentB || !d_latentA || !d_latentB)) return LORDBA_ERR_NULL;
    if (T > 0 && (!x || !g)) return LORDBA_ERR_NULL;
    if ((dx == nullptr) != (dx_base == nullptr)) return LORDBA_ERR_NULL;
    if (t_saved != nullptr && (t_stride < T || t_stride > INT32_MAX)) return LORDBA_ERR_DIM;
    // every pointer aligned to its element; the workspace to 16 bytes (its layout is this library's)
    if (!aligned_to(x, 2) || !aligned_to(g, 2) || !aligned_to(s_in, 2) || !aligned_to(s_out, 2) || !aligned_to(s_rank, 2) ||
        !aligned_to(packedA, 4) || !aligned_to(packedAt, 4) || !aligned_to(packedBt, 4) || !aligned_to(latentA, 4) ||
        !aligned_to(latentB, 4) || !aligned_to(d_s_in, 4) || !aligned_to(d_s_rank, 4) || !aligned_to(d_s_out, 4) ||
        !aligned_to(d_latentA, 4) || !aligned_to(d_latentB, 4) || !aligned_to(workspace, 16) || !aligned_to(t_saved, 4) ||
        !aligned_to(dx_base, 2) || !aligned_to(dx, 2))
        return LORDBA_ERR_ALIGN;
    // The plain matrix-core wgrad and finish kernels need widths that are multiples of 32, 16-byte aligned activations and
    // carriers, and a kept t whose rows reach the padded token count (it is read in whole 32-row steps).
    const bool fast = fast_shape(d_in, d_out) && aligned_to(x, 16) && aligned_to(g, 16) && aligned_to(s_in, 16) && aligned_to(s_out, 16) &&
                      aligned_to(packedA, 16) && aligned_to(packedAt, 16) && aligned_to(dx_base, 16) && aligned_to(dx, 16) &&
                      (t_saved == nullptr || (aligned_to(t_saved, 16) && t_stride % 4 == 0 && t_stride >= (T + 127) / 128 * 128));
    // The same kernels with element-aligned accesses take everything else that has a whole group of 8 columns on either side, with
    // a kept t whose rows reach the padded token count (us, the general kernel's time in brackets: 300 x 1000 -> 3001, r = 12 17.4
    // (362); 600 x 4728 -> 11055, r = 32 37.8 (1902); 4000 x 999 -> 1001, r = 16 21.9 (7178); 64 x 33 -> 17, r = 3 11.1 (19.4).
    const bool any_ok = d_in >= 8 && d_out >= 8 && (t_saved == nullptr || t_stride >= (T + 127) / 128 * 128);
    // Not where a column's r T multiply-adds are so few that one launch which does them one after the other is over before the two
    // launches of the matrix-core path are: the general kernel takes about 6 us and 0.25 (r = 1), 0.4 (3, 4), 0.5 (5), 0.65 (8) more
    // per row, the others about 10.7 whatever the rows (us, matrix-core path in brackets: one row of 33 -> 17, r = 3 6.3 (10.5),
    // 1001 -> 1003, r = 4 8.2 (10.7), 999 -> 12777, r = 8 15.7 (18.4); 5 x 101 -> 65, r = 5 9.2 (10.7) but 9 rows 11.2 (10.8); from
    // r = 9 on it needs twice the registers and loses at one row: 513 -> 515, r = 12 13.0 (11.2)).
    // (One rank and fewer than four rows have to stay among these: row_piece counts on a second row.)
    const bool few = r <= 8 && r * T <= 20;
    const bool general = !fast && (few || !any_ok);
    // Several envelopes: with room for the partial sums of all of them (lordba_backward_multi_workspace_bytes) and at most
    // four rank blocks in all, one wgrad and one finish pass serve every envelope (x and g are read once); otherwise one
    // pass per envelope.
    const int64_t rbe = (r + 15) / 16;
    const bool fused = fast && ell > 1 && ell * rbe <= 4 && workspace_bytes >= make_plan(T, d_in, d_out, r, ell).words * 4;
    const BwdPlan p = make_plan(T, d_in, d_out, r, fused ? ell : 1);
    if (workspace_bytes < p.words * 4) return LORDBA_ERR_WORKSPACE;
    {
        // No output (and not the workspace) may overlap an input or another output; dx on top of dx_base is the one
        // exception and is checked by the forward call below.
        struct Span { const void* p; size_t n; };
        const size_t nx = static_cast<size_t>(T) * d_in * 2, ng = static_cast<size_t>(T) * d_out * 2;
        const size_t nA = static_cast<size_t>(r) * d_in, nB = static_cast<size_t>(d_out) * r;
        const size_t L = static_cast<size_t>(ell);
        const Span outs[] = {{d_s_in, L * d_in * 4}, {d_s_rank, L * r * 4},
                             {d_s_out, L * d_out * 4}, {d_latentA, nA * 4}, {d_latentB, nB * 4},
                             {workspace, p.words * 4}, {dx, dx ? nx : 0}};
        const Span ins[] = {{x, nx}, {g, ng}, {packedA, lordba_packed_words(r, d_in) * 4}, {packedAt, lordba_packed_words(d_in, r) * 4},
                            {packedBt, lordba_packed_words(r, d_out) * 4}, {s_in, L * d_in * 2},
                            {s_rank, L * r * 2}, {s_out, L * d_out * 2}, {latentA, nA * 4},
                            {latentB, nB * 4}, {t_saved, t_saved ? (static_cast<size_t>(ell * r - 1) * t_stride + T) * 4 : 0}};
        auto hit = [](const Span& a, const Span& b) {
            const uintptr_t pa = reinterpret_cast<uintptr_t>(a.p), pb = reinterpret_cast<uintptr_t>(b.p);
            return pa != 0 && pb != 0 && a.n != 0 && b.n != 0 && pa < pb + b.n && pb < pa + a.n;  // (optional arguments may be NULL)
        };
        constexpr int no = sizeof(outs) / sizeof(outs[0]), ni = sizeof(ins) / sizeof(ins[0]);
        for (int i = 0; i < no; ++i) {
            for (int j = 0; j < ni; ++j)
                if (hit(outs[i], ins[j])) return LORDBA_ERR_ALIAS;
            for (int j = i + 1; j < no; ++j)
                if (hit(outs[i], outs[j])) return LORDBA_ERR_ALIAS;
        }
    }
    hipStream_t st = static_cast<hipStream_t>(stream);

    if (T == 0) {  // no token rows: every parameter gradient is zero
        float* outs[5] = {d_s_in, d_s_rank, d_s_out, d_latentA, d_latentB};
        const int64_t ns[5] = {ell * d_in, ell * r, ell * d_out, r * d_in, d_out * r};
        for (int i = 0; i < (with_latents ? 5 : 3); ++i) {
            hipLaunchKernelGGL(bwd_zero_kernel, dim3(static_cast<unsigned>((ns[i] + 255) / 256)), dim3(256), 0, st, outs[i], ns[i]);
            if (hipGetLastError() != hipSuccess) return LORDBA_ERR_LAUNCH;
        }
        return LORDBA_OK;
    }

    float* ws = static_cast<float*>(workspace);
    float* duT = ws + p.off_du;
    float* t_own = ws + p.off_t;
    const _Float16* si = static_cast<const _Float16*>(s_in);
    const _Float16* sr = static_cast<const _Float16*>(s_rank);
    const _Float16* so = static_cast<const _Float16*>(s_out);
    lordba_status s;
    // du of every envelope, and dx = dx_base + g DeltaW^T if wanted (all envelopes at once, one rounding): the forward branch
    // of the transposed adapter (it validates its own arguments); du is that call's rank-r intermediate
    s = lordba_forward_multi_save_t(g, packedBt, packedAt, s_out, s_rank, s_in, dx_base, dx, duT, p.t_pad, T, d_out, d_in, r, ell, stream);
    if (s != LORDBA_OK) return s;
    if (t_saved == nullptr) {
        // t of every envelope: the forward branch of the adapter itself, stopped after its rank-r intermediate.  Its second carrier and
        // s_out are not read: with several envelopes it gets the adapter's own d_out, which the forward that keeps t chooses its number of
        // waves by, so that the sums are the same (packedBt stands in as a carrier of as many bits); with one, and for what the plain
        // matrix-core kernels do not take, d_in (packedAt).
        const bool own = ell > 1 && fast && aligned_to(packedBt, 16);
        s = lordba_forward_multi_save_t(x, packedA, own ? packedBt : packedAt, s_in, s_rank, own ? s_out : s_in, nullptr, nullptr, t_own, p.t_pad,
                                        T, d_in, own ? d_out : d_in, r, ell, stream);
        if (s != LORDBA_OK) return s;
    }
    for (int64_t e = 0; e < (fused ? 1 : ell); ++e) {
        const float* tT = t_saved ? t_saved + e * r * t_stride : t_own + e * r * p.t_pad;
        const int64_t tT_stride = t_saved ? t_stride : p.t_pad;

        BwdArgs a;
        a.x = static_cast<const _Float16*>(x);
        a.g = static_cast<const _Float16*>(g);
        a.pA = packedA;
        a.pBt = packedBt;
        a.s_in = si + e * d_in;
        a.s_rank = sr + e * r;
        a.s_out = so + e * d_out;
        a.latA = latentA;
        a.latB = latentB;
        a.kappa = kappa;
        a.d_s_in = d_s_in + e * d_in;
        a.d_s_rank = d_s_rank + e * r;
        a.d_s_out = d_s_out + e * d_out;
        a.d_latA = d_latentA;
        a.d_latB = d_latentB;
        a.tT = tT;
        a.duT = duT + e * r * p.t_pad;
        a.part = ws + p.off_part;
        a.rank_sums = ws + p.off_rank;
        a.rank_parts = rank_parts(T, p.splits - 1);
        a.rank_tokens = static_cast<int>(rank_span(T, a.rank_parts));   // (whole pieces of four: T + 3 at most)
        a.T = static_cast<int>(T);
        a.d_in = static_cast<int>(d_in);
        a.d_out = static_cast<int>(d_out);
        a.r = static_cast<int>(r);
        a.rp = p.rp;
        a.t_pad = p.t_pad;
        a.t_stride = static_cast<int>(tT_stride);
        a.du_stride = p.t_pad;
        a.nbx = p.nbx;
        a.nbg = p.nbg;
        a.dcols = p.dcols;
        a.tw = p.tw;
        a.splits = p.splits;
        a.waves = p.waves;
        a.accumulate = e > 0 ? 1 : 0;
        a.ell = fused ? static_cast<int>(ell) : 1;
        a.any = fast ? 0 : 1;
        if (general) {
            s = r <= 8 ? launch_general<8>(a, st) : r <= 16 ? launch_general<16>(a, st) : r <= 32 ? launch_general<32>(a, st) : launch_general<64>(a, st);
        } else {
            s = launch_all(a, st);
        }
        if (s != LORDBA_OK) return s;
    }
    return LORDBA_OK;
}

}  // namespace

extern "C" lordba_status lordba_backward(const void* x, const void* g,
                                         const uint32_t* packedA, const uint32_t* packedAt, const uint32_t* packedBt,
                                         const void* s_in, const void* s_rank, const void* s_out,
                                         const float* latentA, const float* latentB, float kappa,
                                         const float* t_saved, int64_t t_stride,
                                         const void* dx_base, void* dx,
                                         float* d_s_in, float* d_s_rank, float* d_s_out,
                                         float* d_latentA, float* d_latentB,
                                         void* workspace, size_t workspace_bytes,
                                         int64_t T, int64_t d_in, int64_t d_out, int64_t r, void* stream) {
    return backward_impl(x, g, packedA, packedAt, packedBt, s_in, s_rank, s_out, latentA, latentB, kappa, t_saved, t_stride, dx_base, dx,
                         d_s_in, d_s_rank, d_s_out, d_latentA, d_latentB, workspace, workspace_bytes, T, d_in, d_out, r, 1, stream);
}

extern "C" lordba_status lordba_backward_multi(const void* x, const void* g,
                                               const uint32_t* packedA, const uint32_t* packedAt, const uint32_t* packedBt,
                                               const void* s_in, const void* s_rank, const void* s_out,
                                               const float* latentA, const float* latentB, float kappa,
                                               const float* t_saved, int64_t t_stride,
                                               const void* dx_base, void* dx,
                                               float* d_s_in, float* d_s_rank, float* d_s_out,
                                               float* d_latentA, float* d_latentB,
                                               void* workspace, size_t workspace_bytes,
                                               int64_t T, int64_t d_in, int64_t d_out, int64_t r, int64_t ell, void* stream) {
    return backward_impl(x, g, packedA, packedAt, packedBt, s_in, s_rank, s_out, latentA, latentB, kappa, t_saved, t_stride, dx_base, dx,
                         d_s_in, d_s_rank, d_s_out, d_latentA, d_latentB, workspace, workspace_bytes, T, d_in, d_out, r, ell, stream);
}

// ---------------------------------------------------------------------------- entry point that allocates nothing ----
// For callers that cannot allocate or pass a workspace: the scratch of the call (rank-r intermediates and partial sums, the
// layout of make_plan) lives in a device array of fixed size that belongs to the library.  Every GPU holds its own copy
// at its own address; in host code the array's name is only a handle, so the address is asked for once per device and
// that pointer is what the kernels get.
static __device__ __align__(256) unsigned char scratch[LORDBA_BACKWARD_NOALLOC_MAX_BYTES];

namespace {
lordba_status noalloc_scratch(void** out) {
    static std::mutex mu;
    static void* ptr[64] = {nullptr};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) { (void)hipGetLastError(); return LORDBA_ERR_NO_DEVICE; }
    if (dev < 0 || dev >= 64) return LORDBA_ERR_NO_DEVICE;
    std::lock_guard<std::mutex> g(mu);
    if (ptr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return LORDBA_ERR_NO_DEVICE;
        }
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return LORDBA_OK;
}
}  // namespace

extern "C" lordba_status lordba_backward_noalloc(const void* x, const void* g,
                                                 const uint32_t* packedA, const uint32_t* packedAt, const uint32_t* packedBt,
                                                 const void* s_in, const void* s_rank, const void* s_out,
                                                 const float* latentA, const float* latentB, float kappa,
                                                 const float* t_saved, int64_t t_stride,
                                                 const void* dx_base, void* dx,
                                                 float* d_s_in, float* d_s_rank, float* d_s_out,
                                                 float* d_latentA, float* d_latentB,
                                                 int64_t T, int64_t d_in, int64_t d_out, int64_t r, void* stream) {
    if (!supported(T, d_in, d_out, r)) return LORDBA_ERR_DIM;
    // the size check comes first: a shape beyond the array is refused whatever else is wrong with the call
    if (make_plan(T, d_in, d_out, r).words * 4 > static_cast<size_t>(LORDBA_BACKWARD_NOALLOC_MAX_BYTES)) return LORDBA_ERR_WORKSPACE;
    void* ws = nullptr;
    const lordba_status s = noalloc_scratch(&ws);
    if (s != LORDBA_OK) return s;
    // Nothing in the scratch has to start at zero: every word a kernel reads was written earlier in the same call.
    return backward_impl(x, g, packedA, packedAt, packedBt, s_in, s_rank, s_out, latentA, latentB, kappa, t_saved, t_stride, dx_base, dx,
                         d_s_in, d_s_rank, d_s_out, d_latentA, d_latentB, ws, LORDBA_BACKWARD_NOALLOC_MAX_BYTES, T, d_in, d_out, r, 1, stream);
}
