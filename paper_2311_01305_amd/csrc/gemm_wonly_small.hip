// Weight-only forward for few tokens (decoding, small batches): y = X_hat W~^T + b straight from the packed codes.
//
// The codes are nearly all the traffic, so they are read once and de-quantised in registers; nothing is written to
// the workspace.  A workgroup of 8 wavefronts owns 16 NT output channels x 16 TT tokens and splits K between its
// wavefronts (the partial sums meet in LDS, in a fixed order), so that even one token spreads over N / 16
// workgroups.  A wavefront works on 256 values of K at a time: per 16 output channels two loads of codes in which
// 8 lanes cover the 128 (INT4) or 96 (INT3) contiguous bytes of a row, and one load of (Step, Z).  The matrix
// operand has the row in the lowest lane bits instead (lane l: channel l % 16, values 32 (l / 16) .. + 31 of 128),
// and loading in that order touches four rows per quad of lanes, which the address unit takes one by one: codes
// and activations therefore pass through a region of LDS private to the wavefront (no barriers).  The product is
// v_mfma_f32_16x16x32_f16, whose two operands may enumerate K in any common order: both use the order in which the
// code fields come out of their packed words.
//
// Reads past an edge repeat the last row or the last values of K (their results are not stored, their activations are zero), so that no
// load sits in a branch of its own.  With more token tiles than channel tiles the codes
// are brought to the activations' natural order instead of the other way round (INT4 / INT3, us on the device with the weight in the
// caches, before -> now: 17 tokens 4096 x 4096 7.2 -> 6.4 / 7.2 -> 6.5, 4096 x 11008 13.7 -> 11.6 / 14.0 -> 12.1; one token 11008 x 4096
// 7.9 -> 7.6 / 8.4 -> 8.2; 16 tokens and 64 within 2 %).  The vector unit has 73 operations there for 32 codes a lane with their scale.
//
// Bound by the read of the codes and, for small layers, by the launch and the round trips to memory (a wavefront asks for one chunk
// ahead).  Measured (INT4, groups of 128, us per call on the device, the same weight every call; before = de-quantising the whole weight and
// a 256 x 256-tiled GEMM; from 64 tokens on also the kernel for some hundred tokens, where it is modelled to take less):
//   tokens          1            16           32           64           128          256
//   4096 x 4096     85.7 ->  4.4  85.8 ->  5.2  86.3 ->  6.9  86.8 ->  8.7  88.2 -> 12.9  87.6 -> 20.9
//   11008 x 4096     100 ->  7.6   101 ->  9.9   101 -> 13.6   102 -> 21.1   103 -> 21.7   103 -> 38.8
//   22016 x 8192     312 -> 22.0   310 -> 26.1   312 -> 37.5   320 -> 39.3   329 -> 69.8   331 ->  129
// (22016 x 8192 at one token: 101 MB of codes and scales, 4.6 TB/s.)  A first form with the operands loaded straight in the matrix
// operand's order, and no pass through LDS, took 6.2 / 13.9 / 42.5 for one token where this one's began with 5.2 / 10.3 / 26.3.
#include "dequant.hpp"
#include "gemm_wonly_small.hpp"

namespace aweq {
namespace wonly {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int kChunk = 256;   // values of K a wavefront takes at a time

// LDS per wavefront: 128 values of RX tokens (256 for RX = 4), 256 codes of 16 NT channels (16 bytes per 32 codes)
constexpr int small_wave_lds(int rx, int nt) { return (rx == 4 ? 4 * 512 : rx * 256) + nt * 16 * 128; }

// RX: tokens of a tile whose activations are loaded: 4, 8, 12, 16, 20, 24 or 32.  What a quad of tokens costs is its load, its way through LDS
// and, with two MFMA tiles of tokens, its share of the operand; left out by a branch around each load instead, as tiles of 16 and 32 once did, the
// compiler waited for more than it needed (us, branches -> this: INT4 6 tokens 4096 x 11008 9.6 -> 8.9, 8 tokens 11008 x 4096 9.8 -> 9.3, 12 tokens
// 8192 x 8192 13.0 -> 12.5, 20 tokens 4096 x 4096 6.5 -> 6.15; INT3 11 tokens 4096 x 4096 5.5 -> 5.2, 17 tokens
// 4096 x 11008 12.5 -> 11.7, 22 tokens 4096 x 2048 5.45 -> 5.35; long rows of many channels, where the codes come at the memory's rate either way, within the
// spread of 2 %: INT4 10 tokens 8192 x 22016 37.8 / 38.2, 12288 x 22016 55.6 / 55.5).  The activations of the second half of a
// chunk are requested ahead of the next codes (loads return in order, and they are needed first).  A chunk more of codes and activations in flight
// gained nothing and its registers cost wavefronts (17 tokens 4096 x 11008 INT3 12.6 -> 13.3, one token 8192 x 8192 9.8 -> 10.9).
// SCALES: kFine: groups that are no multiple of 128 (a lane's 32 codes have one (Step, Z), but the four lanes that share
// 128 values of a channel may differ); kRagged: one (Step, Z) for a row or the tensor, and K ends inside such 128 values
enum { kWhole, kRagged, kFine };
template <int BITS, int RX, int NT, int WAVES, int SCALES, bool OUT_F16>
__global__ __launch_bounds__(WAVES * kWave) void gemm_small_kernel(SmallArgs g)
{
    constexpr int TT = (RX + 15) / 16;
    constexpr bool FINE = SCALES == kFine;
    constexpr int XH = RX == 4 ? 1 : 2;             // activation loads per chunk: whole, or 128 values at a time
    constexpr int XL = RX == 4 ? 2 : RX / 4;        // 16-byte loads of activations per lane and time
    constexpr bool kNatural = TT > NT;              // the operand with fewer tiles is the one that is brought to the other's order
    constexpr bool kCodesLate = RX > 4;
    constexpr int kWords = BITS == 4 ? 4 : 3;
    typedef int Words __attribute__((ext_vector_type(kWords)));
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int r = lane & 15, q = lane >> 4;
    const int64_t n0 = (int64_t)blockIdx.x * (16 * NT), t0 = (int64_t)blockIdx.y * (16 * TT);
    const int K = (int)g.K;
    char* const lx = lds + wave * small_wave_lds(RX, NT);
    char* const lc = lx + (RX == 4 ? 4 * 512 : RX * 256);

    // codes: lane -> row 8 i + lane / 8 of 16, 32 codes lane % 8 of 256.  Rows past the edge re-read the last valid
    // row; their results are never stored.  (32-bit offsets from the tile's first row: 64 rows of K <= 2^20 at most)
    const int c_row = lane >> 3, c_piece = lane & 7;
    const uint32_t code_pitch = (uint32_t)(K >> 3) * BITS;
    const uint8_t* const cbase = g.codes + n0 * code_pitch;
    const int rows_left = (int)min(g.N - n0, (int64_t)(16 * NT)) - 1;
    uint32_t crow[NT][2];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) crow[j][i] = (uint32_t)min(16 * j + 8 * i + c_row, rows_left) * code_pitch;
    // (Step, Z): lane -> row lane / 4 of 16, {Step, Step, Z, Z} of the chunk's first / second 128 values
    const uint32_t* const sbase = ((lane & 2) ? reinterpret_cast<const uint32_t*>(g.zero) : reinterpret_cast<const uint32_t*>(g.step)) +
                                  n0 * g.scale_pitch;
    uint32_t srow[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) srow[j] = (uint32_t)min(16 * j + (FINE ? r : lane >> 2), rows_left) * g.scale_pitch;
    // activations: lane -> token 4 i + lane / 16, 8 values lane % 16 of 128 (RX = 4: the second load is the second 128).  Tokens past the
    // edge re-read the last one; their columns are not stored.
    const _Float16* const xbase = g.X + t0 * g.ldx;
    const int tokens_left = (int)min(g.T - t0, (int64_t)(16 * TT));
    constexpr int XR = RX == 4 ? 1 : XL;
    uint32_t xrow[XR];
#pragma unroll
    for (int i = 0; i < XR; ++i)
        xrow[i] = min((uint32_t)(lane >> 4) * (uint32_t)g.ldx + (uint32_t)(4 * i) * (uint32_t)g.ldx, (uint32_t)(tokens_left - 1) * (uint32_t)g.ldx);

    RawCodes<BITS> rc[NT][2];
    uint32_t sc[NT];
    v4i xr[XL] = {};
    // (past K the last values again: the activations they meet are zero)
    auto load_codes_at = [&](int k) {
        const uint32_t co = (uint32_t)(min(k + c_piece * 32, K - 32) >> 5) * (4 * BITS);
        const uint32_t so = FINE ? 0u : __umulhi((uint32_t)min(k + (lane & 1) * 128, K - 32) >> 4, g.group_magic);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
#pragma unroll
            for (int i = 0; i < 2; ++i) rc[j][i] = load_codes<BITS>(cbase + (crow[j][i] + co));
            sc[j] = FINE ? 0u : sbase[srow[j] + so];
        }
    };
    auto load_x_at = [&](int k) {
        if constexpr (RX == 4) {
            if ((lane >> 4) >= tokens_left) return;   // (a quarter of the lines for one token)
        }
#pragma unroll
        for (int i = 0; i < XL; ++i) {
            const uint32_t xo = (uint32_t)min((RX == 4 ? k + 128 * i : k) + (lane & 15) * 8, K - 8);
            xr[i] = *reinterpret_cast<const v4i*>(xbase + (xrow[RX == 4 ? 0 : i] + xo));
        }
    };

    auto row_of = [&](int i) { return RX - 16 * i < 16 ? min(r, RX - 16 * i - 1) : r; };   // (lanes past the tile's tokens repeat the last one)
    // Four wavefronts keep two sums, of every other chunk each, so that no chain of additions is longer than eight wavefronts' (with one, the error
    // against 64 bits grew from 1.5e-7 to 2.0e-7 at K = 4096)
    constexpr int kSets = WAVES < 8 ? 2 : 1;
    v4f acc[TT][NT], other[kSets == 2 ? TT : 1][kSets == 2 ? NT : 1];
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
            if constexpr (kSets == 2) other[i][j] = acc[i][j];
        }
    auto swap_sets = [&]() {
        if constexpr (kSets == 2) {
#pragma unroll
            for (int i = 0; i < TT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const v4f a = acc[i][j];
                    acc[i][j] = other[i][j];
                    other[i][j] = a;
                }
        }
    };

    // the quad of channels of one token that this thread stores
    constexpr int kTiles = TT * NT;
    static_assert(kTiles <= WAVES, "one quad a thread");
    const int et = wave;
    auto token = [&]() { return t0 + 16 * (et / NT) + (lane & 15); };
    auto channel = [&]() { return n0 + 16 * (et % NT) + 4 * (lane >> 4); };
    auto mine = [&]() { return et < kTiles && token() < g.T && channel() < g.N; };   // N % 4 == 0: all four channels or none
    // up to four tokens its bias is requested ahead of the operands (11008 x 4096, one token, not in a cache 9.5 -> 9.0 us; with
    // more tokens the registers cost a wavefront: 16 tokens 22016 x 8192 34 -> 37.5)
    v4f bias = {0.f, 0.f, 0.f, 0.f};
    if (RX == 4 && g.bias && mine()) bias = *reinterpret_cast<const v4f*>(g.bias + channel());

    // This wavefront's chunks: wave, wave + WAVES, ...  Where rows begin a multiple of 4 KiB apart, all of them lie on the same memory channels at
    // one K, and the workgroups of an XCD begin this round at different places (INT4, us, one / five / 16 tokens: 8192 x 8192 12.05 -> 9.85 /
    // 14.3 -> 11.6 / 15.8 -> 14.0, 4096 x 16384 10.5 -> 9.75 / 12.05 -> 11.65 / 14.8 -> 14.2; elsewhere no gain, and up to 6 % lost where the
    // activations are large: 33 tokens 8192 x 22016 51.5 -> 54.9).
    const int cnt = max(((K + kChunk - 1) / kChunk - wave + WAVES - 1) / WAVES, 0);
    // Held here, all arguments come in one round trip; tiles without branches around their loads otherwise had the pointers in a second one, behind the
    // branch below, 0.15 - 0.25 us of every call (INT4 20 tokens 4096 x 2048 4.60 -> 4.39, 8 tokens 4096 x 4096 5.46 -> 5.31, INT3 17 tokens 1024 x 2048 4.57 -> 4.37)
    asm volatile("" ::"s"(g.X), "s"(g.codes), "s"(g.step), "s"(g.zero), "s"(g.scale_pitch), "s"(g.group_magic));
    int at = code_pitch % 4096 == 0 ? (int)((blockIdx.x / kXcdCount % 16) * (unsigned)cnt / 16u) : 0, kc = (wave + at * WAVES) * kChunk;
    if (cnt > 0) {
        load_codes_at(kc);
        // Codes first: the compiler otherwise puts them behind the addresses of all activations, and a wavefront with one chunk waits for that. (17 - 32 tokens;
        // us, INT3 24 tokens 2048 x 2048 4.68 -> 4.45, INT4 28 tokens 512 x 8192 10.7 -> 10.25; with 16 wavefronts 17 tokens 4096 x 11008 11.8 -> 12.1)
        if constexpr (kNatural && WAVES == 8) __builtin_amdgcn_sched_barrier(0);
        load_x_at(kc);
    }
    for (int left = cnt; left > 0; --left) {
        at = at + 1 == cnt ? 0 : at + 1;
        const int kn = left > 1 ? (wave + at * WAVES) * kChunk : K;   // (K: none)
        uint32_t scc[NT];
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            scc[j] = sc[j];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int row = 8 * i + c_row;
                Words w;   // (INT3: 12 bytes of the 16.  As four registers the compiler waited for the load here, to move it)
#pragma unroll
                for (int e = 0; e < kWords; ++e) w[e] = (int)rc[j][i].w[e];
                *reinterpret_cast<Words*>(lc + j * 2048 + row * 128 + ((c_piece ^ (row & 7)) * 16)) = w;
            }
        }
        wave_lds_fence();
        if (!kCodesLate && kn < K) load_codes_at(kn);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (kc + h * 128 >= K) break;
            if (h < XH) {
#pragma unroll
                for (int i = 0; i < XL; ++i) {
                    const int row = (RX == 4 ? 0 : 4 * i) + (lane >> 4), k = kc + (RX == 4 ? i : h) * 128;
                    if (k + 128 > K && k + (lane & 15) * 8 >= K) xr[i] = v4i{0, 0, 0, 0};
                    *reinterpret_cast<v4i*>(lx + (RX == 4 ? i * 1024 : 0) + row * 256 + (((lane & 15) ^ (row & 15)) * 16)) = kNatural ? xr[i] : pair_order(xr[i]);
                }
                wave_lds_fence();
                const int kx = h + 1 < XH && kc + 128 < K ? kc + 128 : kn;
                if (kx < K) load_x_at(kx);
                // (loads return in order: behind the second half's activations, which are needed first)
                if (kCodesLate && h == 0 && kn < K) load_codes_at(kn);
            }
            // the operand with fewer tiles stays in registers over the loop on the other
            auto frag_x = [&](int i, int d) {
                return __builtin_bit_cast(v8h, *reinterpret_cast<const v4i*>(lx + (RX == 4 ? h * 1024 : i * 4096) + row_of(i) * 256 + (((4 * q + d) ^ row_of(i)) * 16)));
            };
            auto frag_w = [&](int j, uint32_t w[4][4]) {
                const Words cw = *reinterpret_cast<const Words*>(lc + j * 2048 + r * 128 + (((4 * h + q) ^ (r & 7)) * 16));
                RawCodes<BITS> c;
#pragma unroll
                for (int e = 0; e < kWords; ++e) c.w[e] = (uint32_t)cw[e];
                Scale<BITS> s;
                if constexpr (FINE) {
                    const int k = kc + h * 128 + q * 32;
                    const int64_t gi = n0 * g.scale_pitch + srow[j] + (k < K ? __umulhi((uint32_t)k >> 4, g.group_magic) : 0u);
                    s.set(g.step[gi], g.zero[gi]);
                } else {
                    s.set(__uint_as_float((uint32_t)__builtin_amdgcn_ds_bpermute((4 * r + h) * 4, (int)scc[j])),
                          __builtin_amdgcn_ds_bpermute((4 * r + 2 + h) * 4, (int)scc[j]));
                }
                // Past K the weights are zero too: one beyond binary16's range, which stands there again, would make NaN of a zero activation.
                // (Selected in every launch it cost 1 - 3 %; where K is ragged one token 4096 x 4160 4.35 -> 4.40 us, 8 tokens INT3 11008 x 4160 9.5 -> 9.7)
                if (SCALES != kWhole && kc + h * 128 + q * 32 >= K) { s.step = f16x2{(_Float16)0.0f, (_Float16)0.0f}; s.step_f = 0.0f; }
                if (__all(s.packed)) {
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        if constexpr (kNatural) {
                            const v4i o = dequant_word_natural<BITS>(fields_of<BITS>(c, d), s);
#pragma unroll
                            for (int e = 0; e < 4; ++e) w[d][e] = (uint32_t)o[e];
                        } else {
                            dequant8_pairs<BITS>(c, d, s, w[d]);
                        }
                    }
                } else {
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        dequant8_pairs_any<BITS>(c, d, s, w[d]);
                        if constexpr (kNatural) {
                            const v4i o = natural_order(w[d]);
#pragma unroll
                            for (int e = 0; e < 4; ++e) w[d][e] = (uint32_t)o[e];
                        }
                    }
                }
            };
            auto mul = [&](int i, int j, const uint32_t w[4], v8h x) {
                const v4i a = {(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), x, acc[i][j], 0, 0, 0);
            };
            if constexpr (TT <= NT) {
                v8h x[TT][4];
#pragma unroll
                for (int i = 0; i < TT; ++i)
#pragma unroll
                    for (int d = 0; d < 4; ++d) x[i][d] = frag_x(i, d);
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    uint32_t w[4][4];
                    frag_w(j, w);
#pragma unroll
                    for (int d = 0; d < 4; ++d)
#pragma unroll
                        for (int i = 0; i < TT; ++i) mul(i, j, w[d], x[i][d]);
                }
            } else {
                uint32_t w[NT][4][4];
#pragma unroll
                for (int j = 0; j < NT; ++j) frag_w(j, w[j]);
#pragma unroll
                for (int i = 0; i < TT; ++i)
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        const v8h x = frag_x(i, d);
#pragma unroll
                        for (int j = 0; j < NT; ++j) mul(i, j, w[j][d], x);
                    }
            }
            wave_lds_fence();   // this chunk's reads stay ahead of the next one's writes
        }
        kc = kn;
        swap_sets();
    }

    // register v of lane l is output channel 4 (l / 16) + v of the 16, token l % 16
    float* const red = reinterpret_cast<float*>(lds);   // [set][wave][TT NT][lane][4]
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            *reinterpret_cast<v4f*>(red + ((wave * kTiles + i * NT + j) * kWave + lane) * 4) = acc[i][j];
            if constexpr (kSets == 2) *reinterpret_cast<v4f*>(red + (((WAVES + wave) * kTiles + i * NT + j) * kWave + lane) * 4) = other[i][j];
        }
    __syncthreads();
    if (!mine()) return;
    const int64_t t = token(), n = channel();
    v4f o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < WAVES * kSets; ++w) o += *reinterpret_cast<const v4f*>(red + ((w * kTiles + et) * kWave + lane) * 4);
    if (g.bias) o += RX == 4 ? bias : *reinterpret_cast<const v4f*>(g.bias + n);
    if constexpr (OUT_F16) {
        typedef _Float16 h4 __attribute__((ext_vector_type(4)));
        *reinterpret_cast<h4*>(reinterpret_cast<_Float16*>(g.out) + t * g.ldo + n) =
            h4{(_Float16)o[0], (_Float16)o[1], (_Float16)o[2], (_Float16)o[3]};
    } else {
        *reinterpret_cast<v4f*>(reinterpret_cast<float*>(g.out) + t * g.ldo + n) = o;
    }
}

template <int BITS, int RX, int NT, int WAVES>
static int launch_tile(const SmallArgs& g, int scales, bool out_f16, hipStream_t st)
{
    constexpr int TT = (RX + 15) / 16;
    static_assert(RX == 4 || RX % 16 == 0 || RX < 32, "a tile that is not whole holds all tokens of the call");
    const dim3 grid((unsigned)cdiv(g.N, 16 * NT), (unsigned)cdiv(g.T, 16 * TT));
    constexpr int work = WAVES * small_wave_lds(RX, NT), red = (WAVES < 8 ? 2 : 1) * WAVES * TT * NT * kWave * 16;
    constexpr int lds = work > red ? work : red;
#define AWEQ_SF(S) (out_f16 ? reinterpret_cast<const void*>(gemm_small_kernel<BITS, RX, NT, WAVES, S, true>) \
                            : reinterpret_cast<const void*>(gemm_small_kernel<BITS, RX, NT, WAVES, S, false>))
    const void* fn = scales == kFine ? AWEQ_SF(kFine) : scales == kRagged ? AWEQ_SF(kRagged) : AWEQ_SF(kWhole);
#undef AWEQ_SF
    int dev = 0, cus = 0;
    if (lds > 65536 && (device_cus(dev, cus) != AWEQ_OK || raise_lds_limit(fn, dev, lds) != AWEQ_OK)) return AWEQ_ERR_LAUNCH;
    void* args[] = {const_cast<SmallArgs*>(&g)};
    if (hipLaunchKernel(fn, grid, dim3(WAVES * kWave), args, lds, st) != hipSuccess) return AWEQ_ERR_LAUNCH;
    return launch_status();
}

SmallPlan plan_small(int64_t T, int64_t N)
{
    // Up to 16 tokens the pass is a read of the codes: 16 channels per workgroup until those workgroups fill the chip
    // 1.5 times over, then 32, which read the tokens half as often (us with 16 / 32 channels: one token 4096 x 4096 4.4 / 5.9, 8192 x 8192
    // 9.3 / 10.3, 22016 x 8192 the same; four tokens 22016 x 8192 23.7 / 22.3; 8 tokens 12800 x 8192 19.5 / 17.4; 16 tokens 16384 x 4096
    // 13.7 / 11.5, but 8192 x 8192 13.2 / 11.8, which the line does not see; 64 channels lose everywhere).  Nothing else comes near.
    if (T <= 16) return {N > 12288 ? 2 : 1, 0.0};
    // More tokens, 32 per workgroup: as many channels as give the fewest rounds of workgroups, each weighted with what a
    // round was measured to take when a load sat in a branch (8192 x 8192, 17 tokens, us: 19 for 512 workgroups of 16 channels, two per
    // compute unit, 14 for 256; 17.5 for 32 channels and 27 for 64, one per compute unit).  Now a compute unit's first, second, third and fourth
    // workgroup of 16 channels take 8.3, 7.6, 6.4 and 6.8, one of 32 channels 13 - 14, of 64 channels 21 and 27 (17 to 20 tokens; 21 to 24 up to a tenth more).
    // The line stays: over 1742 shapes of 17 to 24 tokens its choice takes 0.5 % more than the fastest form, in 168 more than 3 % (most: INT3 of 8200 to
    // 12288 and 16400 to 20000 channels, where 16 a workgroup are the faster form, 18 tokens 19396 x 8448 46.0 / 41.6); weights fitted to these times were 0.2 %
    // better in the mean and in 89 shapes 2 - 13 % slower (22 tokens 12328 x 8320 24.2 -> 27.2).  64 tokens per workgroup gained nothing
    // (4096 x 4096 10.4 us in 32s, 14.0 in 64s; 22016 x 8192 76 / 75).
    const int64_t tm = cdiv(T, 32), w1 = cdiv(N, 16) * tm, w2 = cdiv(N, 32) * tm, w4 = cdiv(N, 64) * tm;
    const double c1 = w1 <= 256 ? 14.0 : 19.0 * (double)cdiv(w1, 512), c2 = 17.5 * (double)cdiv(w2, 256), c4 = 27.0 * (double)cdiv(w4, 256);
    if (c1 <= c2 && c1 <= c4) return {1, c1};
    return c2 <= c4 ? SmallPlan{2, c2} : SmallPlan{4, c4};
}

template <int BITS>
static int launch_bits(const SmallArgs& g, int scales, int nt, bool out_f16, hipStream_t st)
{
    // Long rows on at most one workgroup per compute unit: K split between 16 wavefronts instead of 8, from two chunks a wavefront on (us, INT4,
    // 8 -> 16: one token 1024 x 22016 12.0 -> 10.7, 4096 x 11008 7.6 -> 7.1, 2048 x 8192 6.1 -> 5.9, 4096 x 4096 the same; 16 tokens 1024 x 22016
    // 17.2 -> 14.8, but 2048 x 8192 8.4 -> 8.5)
    const bool lone = cdiv(g.N, 16) <= 256;
    // 513 to 768 workgroups (to 1024 of up to four tokens) of short rows: four wavefronts, of which all workgroups are resident at a time; eight
    // take 512 of them, and the rest wait (us, INT4, 8 -> 4: one token 11008 x 4096 8.65 -> 8.4, 12288 x 2048 5.35 -> 4.9, 8704 x 1024 4.45 -> 3.65,
    // 16384 x 4096 (32 channels a workgroup before) 10.25 -> 10.1; 6 tokens 8704 x 4096 9.95 -> 9.2, 16 tokens 11008 x 4096 11.0 -> 10.8; but one
    // token 11008 x 11008 15.8 -> 16.5, INT3 16 tokens 11008 x 5120 12.6 -> 12.9, 6 tokens 16384 x 4096 11.4 -> 11.7)
#define AWEQ_ST(RX, NT, WAVES) launch_tile<BITS, RX, NT, WAVES>(g, scales, out_f16, st)
#define AWEQ_ST16(NT, WAVES) (g.T <= 8 ? AWEQ_ST(8, NT, WAVES) : g.T <= 12 ? AWEQ_ST(12, NT, WAVES) : AWEQ_ST(16, NT, WAVES))
    if (g.T <= 16 && cdiv(g.N, 16) > 512 && g.N <= (g.T <= 4 ? 16384 : 12288) && g.K <= (BITS == 4 ? 8192 : 4096))
        return g.T <= 4 ? AWEQ_ST(4, 1, 4) : AWEQ_ST16(1, 4);
    if (g.T <= 4) {
        if (nt == 2) return AWEQ_ST(4, 2, 8);
        return lone && g.K >= 8192 ? AWEQ_ST(4, 1, 16) : AWEQ_ST(4, 1, 8);
    }
    if (g.T <= 16) {
        if (nt == 2) return AWEQ_ST16(2, 8);
        if (lone && g.K >= 16384) return AWEQ_ST16(1, 16);
        return AWEQ_ST16(1, 8);
    }
    // 17 to 24 tokens on at most one workgroup per compute unit: 16 wavefronts from one chunk a wavefront on (us, 8 -> 16: INT3 17 tokens
    // 4096 x 11008 12.6 -> 11.7, INT4 18 tokens 1024 x 4096 6.0 -> 5.8, 24 tokens 4096 x 11008 12.95 -> 12.6; half a chunk each INT3 22 tokens
    // 4096 x 2048 4.55 -> 4.75; 32 tokens take all registers: 4096 x 4096 7.6 -> 8.05)
    const bool many = nt == 1 && lone && g.K >= 16 * kChunk;
    if (g.T <= 24) {
        if (many) return g.T <= 20 ? AWEQ_ST(20, 1, 16) : AWEQ_ST(24, 1, 16);
        if (nt == 1) return g.T <= 20 ? AWEQ_ST(20, 1, 8) : AWEQ_ST(24, 1, 8);
        if (nt == 2) return AWEQ_ST(24, 2, 8);
        // (a quad of tokens less, us: INT3 17 tokens 12800 x 2048 8.7 -> 8.5, 11008 x 4096 14.65 -> 14.1, 16384 x 4096 16.0 -> 15.6; INT4 within 1 %)
        if constexpr (BITS == 3) { if (g.T <= 20) return AWEQ_ST(20, 4, 8); }
        return AWEQ_ST(24, 4, 8);
    }
    return nt == 1 ? AWEQ_ST(32, 1, 8) : nt == 2 ? AWEQ_ST(32, 2, 8) : AWEQ_ST(32, 4, 8);
#undef AWEQ_ST16
#undef AWEQ_ST
}

int launch_small(const SmallArgs& g, int bits, int group, const SmallPlan& p, bool out_f16, hipStream_t st)
{
    const int scales = group > 0 && group % 128 != 0 ? kFine : g.K % 128 != 0 ? kRagged : kWhole;
    return bits == 4 ? launch_bits<4>(g, scales, p.nt, out_f16, st) : launch_bits<3>(g, scales, p.nt, out_f16, st);
}

}  // namespace wonly
}  // namespace aweq
