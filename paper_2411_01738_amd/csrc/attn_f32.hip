// float32 attention (chunk attention with O and LSE, and the fused PipeFusion
// patch step) with float32 products throughout, on the matrix cores.
//
// What bounds it: the float32 matrix rate, 64 operations per clock and SIMD
// (157 TFLOP/s; v_mfma_f32_32x32x2_f32 takes 64 clocks).  A 32 x 32 tile of
// scores costs 2 * d/2 products (4096 clocks at d = 64) against about 500
// clocks of softmax, most of which issues between the products.  B = 2, 16
// heads of 72, 1024 queries over 1024 keys takes 94 us (102 TFLOP/s, of 154
// that a large float32 matrix product reaches); the matrix cores are busy for
// 67 us of them.  One query per lane with vector FMAs, as this kernel did
// before, took 789 us.
//
// Work decomposition: one workgroup = QB blocks of 32 query rows x KS waves
// that split every tile of 32 KS keys between them; the KS waves keep
// separate running (max, sum, output), merged through LDS at the end.
//   * S^T = K Q^T: K rows come from LDS (global loads with an LDS
//     destination, two stages, 16-byte chunks XOR-swizzled by row so that the
//     16-byte operand reads meet no bank conflict), Q rows sit in registers.
//     The contraction order is free as long as both operands agree: lane
//     half hf takes dims hf*d/2 .., so one 16-byte read feeds four products.
//   * O^T = V^T P^T: the accumulator layout of S^T (lane: one query, 16 keys)
//     is the operand layout of P^T as it stands; V rows go from memory
//     straight to registers (a wave's load of one k-step is two whole rows),
//     issued between the products of the scores.
//   * d = 72: dims 64..71 run as one 16-row block on
//     v_mfma_f32_16x16x4_f32, the weights regrouped by v_permlane16_swap.
#include "kernels.h"

#include <math.h>

#include <type_traits>

namespace xdit {
namespace {

#include "attn_common.h"

constexpr int kKT = 32;  // keys per wave and tile

struct F32Args {
    const float* q;
    const float* k;
    const float* v;
    const float* fk;
    const float* fv;
    float* wk;
    float* wv;
    float* out;
    float* lse;
    int B, H, Nq, Nk, q_tiles;
    int off0, len0, off1, len1;  // fresh ranges (fresh rows: range 0's, then range 1's)
    int sa0, sn0, sa1, sn1;      // tiles [sa, sa + sn) hold rows of fresh range 0 / 1
    float scale;
    int accum;  // merge into the running (out, lse) instead of overwriting them
};

template <int D, int QB_, int KS_>
struct FCfg {
    static constexpr int QB = QB_, KS = KS_;
    static constexpr int NW = QB * KS;
    static constexpr int THREADS = 64 * NW;
    static constexpr int BM = 32 * QB;            // query rows per workgroup
    static constexpr int BN = kKT * KS;           // keys per tile
    static constexpr int CH = D / 4;              // 16-byte chunks per row
    static constexpr int ROWB = 4 * D;            // bytes per row in LDS
    static constexpr int STAGE = BN * ROWB;       // one K tile
    static constexpr int DMA_PER_TILE = STAGE / 1024;
    static constexpr int DMA_PER_WAVE = (DMA_PER_TILE + NW - 1) / NW;
    static constexpr int DBLK = D / 32;           // 32-row blocks of O^T
    static constexpr bool TAIL = D % 32 != 0;     // d = 72: dims 64..71
    static constexpr int KQ = D / 8;              // 16-byte operand reads per lane and tile
    static constexpr int NG = 4 * DBLK;           // groups of 4 output registers
    // V k-steps held at a time: all of a tile's, or a quarter (256-register budget)
    static constexpr int VSTEPS = D > 96 ? 4 : 16;
    // exchange slot of a wave: max, sum, output registers (lane-major)
    static constexpr int XSLOT = 64 * (2 + 4 * NG + (TAIL ? 8 : 0));
    static constexpr int X_BYTES = KS > 1 ? 4 * NW * XSLOT : 0;
    static constexpr int LDS_BYTES = 2 * STAGE > X_BYTES ? 2 * STAGE : X_BYTES;
    // Logical chunk c of row r sits in slot c ^ swz(r).  Sixteen lanes read
    // the same logical chunk of 16 consecutive rows in one cycle: rows of 64
    // or 128 floats start on the same bank, so the slots must differ in the
    // row's low four bits; rows of 72 floats are 8 banks apart, which leaves
    // rows r and r + 8 on the same banks unless their slots differ by one.
    __device__ static constexpr int swz(int r) { return D == 72 ? (r >> 3) & 1 : r & 15; }
    static_assert(D == 64 || D == 72 || D == 128, "head dims");
    static_assert(STAGE % 1024 == 0, "tiles are whole 64-lane loads");
    static_assert(LDS_BYTES <= kLdsBytes, "LDS budget");
};

constexpr float kLog2e = 1.4426950408889634f;
__device__ __forceinline__ float exp_b2(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }

__device__ __forceinline__ void vload(Rsrc r, uint32_t off, float (&x)[1]) {
    x[0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ void vload(Rsrc r, uint32_t off, float (&x)[2]) {
    const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
    x[0] = __uint_as_float(w[0]);
    x[1] = __uint_as_float(w[1]);
}
__device__ __forceinline__ void vload(Rsrc r, uint32_t off, float (&x)[4]) {
    const u32x4 w = bload(r, off);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = __uint_as_float(w[e]);
}

// 16 bytes of running output merged into y by weight w (rows of a ring step)
__device__ __forceinline__ void store_row4(float* dst, f32x4 y, float w_prev) {
    if (w_prev != 0.f) {
        const f32x4 x = *(const f32x4*)dst;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = __builtin_fmaf(w_prev, x[e], y[e]);
    }
    *(f32x4*)dst = y;
}

// Two waves per SIMD: two workgroups of 4 waves, or one of 8; the K stages of
// four waves at d = 128 leave room for one workgroup of 4.
template <int D, int QB, int KS, bool PATCH>
__global__ __launch_bounds__(64 * QB * KS, (QB * KS == 4 && KS * D > 320 ? 1 : 2)) void attn_f32_kernel(F32Args a) {
    using C = FCfg<D, QB, KS>;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[C::LDS_BYTES];
    constexpr int DBLK = C::DBLK;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c = lane & 31, hf = lane >> 5;
    const int qb = wave % QB, kh = wave / QB;  // query block, key split
    const int logical = xcd_remap(blockIdx.x, gridDim.x);
    const int qt = logical % a.q_tiles, bh = logical / a.q_tiles;
    const int hh = bh % a.H, b = bh / a.H;
    const uint32_t rowb = (uint32_t)a.H * D * 4;
    const uint32_t headb = (uint32_t)hh * D * 4;
    const int64_t rs = (int64_t)a.H * D, headoff = (int64_t)hh * D;
    const int F = a.len0 + a.len1;  // fresh rows

    const float* kbase = a.k + (int64_t)b * a.Nk * rs + headoff;
    const float* vbase = a.v + (int64_t)b * a.Nk * rs + headoff;
    const float* fkbase = PATCH ? a.fk + (int64_t)b * F * rs + headoff : nullptr;
    const float* fvbase = PATCH ? a.fv + (int64_t)b * F * rs + headoff : nullptr;
    // rows row0 .. rows-1 of this head (none if row0 >= rows); rows past the end read as zero
    auto rows_rsrc = [&](const float* base, int row0, int rows) -> Rsrc {
        return rsrc(base + (int64_t)row0 * rs, rows > row0 ? (uint32_t)(rows - row0) * rowb - headb : 0u);
    };

    // Q rows as B operands: lane (query c, half hf) holds dims hf*D/2 ..
    const int qrow = qt * C::BM + qb * 32 + c;
    const bool qvalid = qrow < a.Nq;
    f32x4 qf[C::KQ];
    {
        const Rsrc rq = rows_rsrc(a.q + (int64_t)b * a.Nq * rs + headoff, qt * C::BM, a.Nq);
#pragma unroll
        for (int j = 0; j < C::KQ; ++j)
            qf[j] = __builtin_bit_cast(f32x4, bload(rq, (uint32_t)(qb * 32 + c) * rowb + 16 * (hf * C::KQ + j)));
    }

    // K tile loads: load n of this wave fills 64 chunks of a stage
    uint32_t dma_off[C::DMA_PER_WAVE];
#pragma unroll
    for (int n = 0; n < C::DMA_PER_WAVE; ++n) {
        const int p = 64 * (wave + n * C::NW) + lane, r = p / C::CH;
        dma_off[n] = (uint32_t)r * rowb + 16 * ((p % C::CH) ^ C::swz(r));
    }
    // Where tile t's rows come from: 0 = buffer (or chunk), 1 / 2 = wholly
    // fresh range 0 / 1, 3 = straddles a range edge.
    auto source = [&](int t) -> int {
        if (!PATCH || ((unsigned)(t - a.sa0) >= (unsigned)a.sn0 && (unsigned)(t - a.sa1) >= (unsigned)a.sn1)) return 0;
        const int lo = t * C::BN, hi = min(lo + C::BN, a.Nk);
        if (a.off0 <= lo && hi <= a.off0 + a.len0) return 1;
        if (a.off1 <= lo && hi <= a.off1 + a.len1) return 2;
        return 3;
    };
    // the fresh row that holds buffer row j, or -1
    auto fresh_row = [&](int j) -> int {
        if ((unsigned)(j - a.off0) < (unsigned)a.len0) return j - a.off0;
        if ((unsigned)(j - a.off1) < (unsigned)a.len1) return a.len0 + j - a.off1;
        return -1;
    };
    // resource of tile t's rows for sources 0..2
    auto tile_rsrc = [&](int src, int t, const float* base, const float* fbase) -> Rsrc {
        const int lo = t * C::BN;
        if (!PATCH || src == 0) return rows_rsrc(base, lo, a.Nk);
        return src == 1 ? rows_rsrc(fbase, lo - a.off0, a.len0) : rows_rsrc(fbase, a.len0 + lo - a.off1, F);
    };
    auto load_k = [&](int t, int s) {
        unsigned char* dst = lds + s * C::STAGE;
        const int src = source(t);
        if (src != 3) {
            const Rsrc r = tile_rsrc(src, t, kbase, fkbase);
#pragma unroll
            for (int n = 0; n < C::DMA_PER_WAVE; ++n) {
                const int ins = wave + n * C::NW;
                if (C::DMA_PER_TILE % C::NW == 0 || ins < C::DMA_PER_TILE) dma16(r, dst + 1024 * ins, dma_off[n]);
            }
            return;
        }
        const int lo = t * C::BN;
        const Rsrc rk = rows_rsrc(kbase, lo, a.Nk), fk = rows_rsrc(fkbase, 0, F);
#pragma unroll
        for (int n = 0; n < C::DMA_PER_WAVE; ++n) {
            const int ins = wave + n * C::NW;
            if (C::DMA_PER_TILE % C::NW == 0 || ins < C::DMA_PER_TILE) {
                const int r = (64 * ins + lane) / C::CH, fr = fresh_row(lo + r);
                if (fr >= 0) dma16(fk, dst + 1024 * ins, dma_off[n] + (uint32_t)(fr - r) * rowb);
                else dma16(rk, dst + 1024 * ins, dma_off[n]);
            }
        }
    };
    // V operands of this wave's 32 keys: k-step i is key 8(i/4) + 4hf + i%4
    // (the order of the weights), vv[i][db] dim DBLK c + db, so that one load
    // brings a lane its dims of all blocks; the tail's k-step p holds dims
    // 64 + lane%16 of the keys its regrouped weights hold, row 8(p/2) +
    // 2(p%2) + trow.
    const int grp = lane >> 4, l16 = lane & 15;
    auto vkey = [&](int i) { return kh * kKT + 8 * (i >> 2) + 4 * hf + (i & 3); };
    const int trow = (grp & 1) + 4 * (grp >> 1);
    const uint32_t vbyte = 4 * DBLK * c, voff = (uint32_t)(4 * hf) * rowb + vbyte;
    const uint32_t tbyte = 4 * (64 + l16), toff = (uint32_t)trow * rowb + tbyte;
    constexpr int NTP = C::TAIL ? 8 : 0;
    constexpr int VN = C::VSTEPS;
    // what tile t's V loads share: buffer row j of the tile is source row
    // j - row0 of r (src 0..2; r ends with the source), or each lane's row
    // has a source of its own (src 3: r the buffer, fr the fresh rows)
    struct VTile {
        Rsrc r, fr;
        int src, row0;
        uint32_t vo, to;
    };
    // source(), for this wave's 32 rows alone
    auto v_source = [&](int lo) -> int {
        if (!PATCH) return 0;
        const int hi = min(lo + kKT, a.Nk);
        if (a.off0 <= lo && hi <= a.off0 + a.len0) return 1;
        if (a.off1 <= lo && hi <= a.off1 + a.len1) return 2;
        const bool in0 = a.len0 > 0 && lo < a.off0 + a.len0 && a.off0 < hi;
        const bool in1 = a.len1 > 0 && lo < a.off1 + a.len1 && a.off1 < hi;
        return in0 || in1 ? 3 : 0;
    };
    auto v_tile = [&](int t) -> VTile {
        VTile x;
        x.row0 = t * C::BN + kh * kKT;  // this wave's first row of the tile
        x.src = v_source(x.row0);
        const bool buf = x.src == 0 || x.src == 3;
        const int shift = buf ? 0 : (x.src == 1 ? -a.off0 : a.len0 - a.off1);
        x.r = rows_rsrc(buf ? vbase : fvbase, x.row0 + shift, buf ? a.Nk : (x.src == 1 ? a.len0 : F));
        x.fr = PATCH ? rows_rsrc(fvbase, 0, F) : x.r;
        // opaque per tile, so that the offsets of the k-steps are derived
        // from it as needed rather than each kept in a register of its own
        x.vo = voff;
        x.to = toff;
        asm volatile("" : "+v"(x.vo), "+v"(x.to));
        return x;
    };
    // V operands of k-step i (and of the tail's k-step i/2 with the even ones)
    auto load_v = [&](const VTile& x, int i, float (&vv)[DBLK], float& vt) {
        const int ri = 8 * (i >> 2) + (i & 3);
        const uint32_t ro = (uint32_t)ri * rowb;
        const bool tail = C::TAIL && i % 2 == 0;
        float tl[1];
        if (!PATCH || x.src != 3) {
            vload(x.r, x.vo + ro, vv);
            if (tail) {
                vload(x.r, l16 < 8 ? x.to + ro : kOOB, tl);
                vt = tl[0];
            }
            return;
        }
        const int fr = fresh_row(x.row0 + ri + 4 * hf);
        if (fr >= 0) vload(x.fr, (uint32_t)fr * rowb + vbyte, vv);
        else vload(x.r, x.vo + ro, vv);
        if (tail) {
            const int ft = fresh_row(x.row0 + ri + trow);
            if (ft >= 0) vload(x.fr, l16 < 8 ? (uint32_t)ft * rowb + tbyte : kOOB, tl);
            else vload(x.r, l16 < 8 ? x.to + ro : kOOB, tl);
            vt = tl[0];
        }
    };

    f32x16 o[DBLK];
#pragma unroll
    for (int db = 0; db < DBLK; ++db) o[db] = f32x16{};
    f32x4 ot[2] = {f32x4{}, f32x4{}};  // tail: queries 16h + lane%16, dims 64 + 4(lane/16) + e
    float m = -INFINITY, l = 0.f;      // of this wave's keys; l: this lane's share

    const uint32_t lds_u32 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
    const int krow = kh * kKT + c;
    const uint32_t kaddr = lds_u32 + krow * C::ROWB;
    const int ntiles = (a.Nk + C::BN - 1) / C::BN;
    // this wave's keys of tile t: [first_key(t), ...); a wave past the end has none
    auto first_key = [&](int t) { return t * C::BN + kh * kKT; };
    // the tile loads this wave issued have landed, then everybody's
    auto meet = [&]() {
        wait_vmem<0>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    // Scores of tile t into sn (QK; raw, before the scale), with the softmax
    // of the previous tile's scores sc between the products (SM), and with(n)
    // after product n: a product holds the matrix pipe for 64 clocks, under
    // which a dozen VALU instructions of the same wave issue.  Left to itself
    // each phase of the two waves of a SIMD met the same phase of the other
    // (they share the pipe evenly, so they reach the softmax together).
    auto phase = [&](int t, f32x16& sc, f32x16& sn, auto qk_c, auto sm_c, auto&& with) {
        constexpr bool QK = decltype(qk_c)::value, SM = decltype(sm_c)::value;
        constexpr int NS = 4 * C::KQ;
        static_assert(NS >= 24, "one piece of softmax per product");
        const uint32_t ka0 = kaddr + (t & 1) * C::STAGE;
        auto read_k = [&](int j) { return lds_ld<f32x4>(ka0 + 16 * ((hf * C::KQ + j) ^ C::swz(krow))); };
        f32x4 ka = {}, kn = {};
        if constexpr (QK) {
            sn = f32x16{};
            ka = read_k(0);
        }
        float mt = -INFINITY, ms = 0.f;
        static_for<0, NS>([&](auto nc) {
            constexpr int n = decltype(nc)::value;
            if constexpr (QK) {
                // the next operand's read goes ahead of this one's products
                if constexpr (n % 4 == 0) kn = n + 4 < NS ? read_k(n / 4 + 1) : ka;
                sn = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[n % 4], qf[n / 4][n % 4], sn, 0, 0, 0);
                if constexpr (n % 4 == 3) ka = kn;
            }
            with(nc);
            if constexpr (SM) {
                if constexpr (n < 2) {
#pragma unroll
                    for (int i = 8 * n; i < 8 * n + 8; ++i) mt = fmaxf(mt, sc[i]);
                } else if constexpr (n == 2) {
                    mt = halves_max(mt) * a.scale;
                    // the reference max is raised only when a row's max exceeds
                    // it by more than 2^8 in weight: rescales are rare, and
                    // float32 sums lose nothing by larger weights
                    if (__builtin_amdgcn_ballot_w64(mt > m + kRescaleLog2 / kLog2e) != 0) {
                        const float m_new = fmaxf(m, mt);
                        // -inf only while no finite score was seen (nothing accumulated)
                        const float alpha = m_new == -INFINITY ? 1.f : exp_b2(m - m_new);
                        m = m_new;
                        l *= alpha;
#pragma unroll
                        for (int db = 0; db < DBLK; ++db) o[db] *= alpha;
                        if constexpr (C::TAIL) {
                            ot[0] *= __shfl(alpha, l16);
                            ot[1] *= __shfl(alpha, 16 + l16);
                        }
                    }
                    ms = m == -INFINITY ? 0.f : m;
                } else if constexpr (n >= 4 && n < 22) {
                    // weight i = n - 4 in three steps, one product apart, so
                    // that no step waits for the one before it
                    constexpr int i = n - 4;
                    if constexpr (i >= 2) l += sc[i - 2];
                    if constexpr (i >= 1 && i < 17) {
                        sc[i - 1] = __builtin_amdgcn_exp2f(sc[i - 1]);
                        asm volatile("" : "+v"(sc[i - 1]));  // here, not at its use
                    }
                    if constexpr (i < 16) {
                        // one rounding: s * scale - max
                        sc[i] = __builtin_fmaf(sc[i], a.scale, -ms) * kLog2e;
                        asm volatile("" : "+v"(sc[i]));
                    }
                }
            }
            if constexpr (QK && SM) __builtin_amdgcn_sched_barrier(0);
        });
    };
    // keys past the end of a ragged last tile
    auto mask = [&](int t, f32x16& s) {
        if (first_key(t) + kKT > a.Nk) {
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (t * C::BN + vkey(i) >= a.Nk) s[i] = -INFINITY;
        }
    };
    using T_ = std::true_type;
    using F_ = std::false_type;
    // Iteration t: the scores of tile t+1 under the softmax of tile t, then
    // PV of tile t.  K tile t+1 has landed when it starts; the stage of tile
    // t, whose scores every wave has, takes tile t+2.  NEXT: this wave has
    // keys in tile t+1.
    f32x16 sc = {};
    auto iteration = [&](int t, auto next_c) {
        constexpr bool NEXT = decltype(next_c)::value;
        if (NEXT && t + 2 < ntiles) load_k(t + 2, t & 1);
        // V k-steps go out one per two products, so that their issue hides
        // under the products too; at d = 128 they load in groups, the next
        // group under this one's products
        const VTile x = v_tile(t);
        constexpr int VG = 16 / VN;
        float vv[VG > 1 ? 2 : 1][VN][DBLK], vt[NTP > 0 ? NTP : 1];
        f32x16 sn;
        phase(t + 1, sc, sn, next_c, T_{}, [&](auto nc) {
            constexpr int n = decltype(nc)::value;
            if constexpr (n % 2 == 0 && n / 2 < VN) load_v(x, n / 2, vv[0][n / 2], vt[NTP > 0 ? n / 4 : 0]);
        });
        static_for<0, 16>([&](auto ic) {
            constexpr int i = decltype(ic)::value, g = i / VN;
            if constexpr (g + 1 < VG) load_v(x, i + VN, vv[(g + 1) % 2][i % VN], vt[0]);
            if constexpr (VG > 1) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int db = 0; db < DBLK; ++db)
                o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[g % 2][i % VN][db], sc[i], o[db], 0, 0, 0);
        });
        if constexpr (C::TAIL) {
            // permlane16_swap of k-steps 2p, 2p+1 gives the 16x16x4
            // operands of queries 0..15 and 16..31: lane group g holds
            // k-step 2p + (g & 1), half g >> 1
#pragma unroll
            for (int p = 0; p < 8; ++p) {
                const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(sc[2 * p]),
                                                                __float_as_uint(sc[2 * p + 1]), false, false);
                ot[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(vt[p], __uint_as_float(r[0]), ot[0], 0, 0, 0);
                ot[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(vt[p], __uint_as_float(r[1]), ot[1], 0, 0, 0);
            }
        }
        if constexpr (NEXT) {
            sc = sn;
            mask(t + 1, sc);
        }
        meet();
    };
    // tiles in which this wave has keys: all, or all but the last one (every
    // wave passes ntiles + 2 barriers)
    const int mine = first_key(ntiles - 1) < a.Nk ? ntiles : ntiles - 1;
    if (ntiles > 0) load_k(0, 0);
    if (ntiles > 1) load_k(1, 1);
    // Patch: this workgroup's share of the fresh rows goes into the buffer
    // while the first tiles load (nothing here reads the buffer's fresh rows;
    // after the sweep the copy had cost a 64-row patch 2 of 12 us).
    if constexpr (PATCH) {
        constexpr int CU = 4;  // 16-byte chunks per lane and batch
        const int r0 = (int)((int64_t)F * qt / a.q_tiles), r1 = (int)((int64_t)F * (qt + 1) / a.q_tiles);
        const int n = (r1 - r0) * C::CH;
        float* wk = a.wk + (kbase - a.k);
        float* wv = a.wv + (vbase - a.v);
        for (int e0 = tid; e0 < n; e0 += CU * C::THREADS) {
            f32x4 ck[CU], cv[CU];
            int64_t to[CU];
#pragma unroll
            for (int u = 0; u < CU; ++u) {
                const int e = min(e0 + u * C::THREADS, n - 1);  // past the share: its last chunk again
                const int fr = r0 + e / C::CH, cc = 4 * (e % C::CH);
                to[u] = (int64_t)(fr < a.len0 ? a.off0 + fr : a.off1 + fr - a.len0) * rs + cc;
                ck[u] = *(const f32x4*)(fkbase + (int64_t)fr * rs + cc);
                cv[u] = *(const f32x4*)(fvbase + (int64_t)fr * rs + cc);
            }
#pragma unroll
            for (int u = 0; u < CU; ++u) {
                *(f32x4*)(wk + to[u]) = ck[u];
                *(f32x4*)(wv + to[u]) = cv[u];
            }
        }
    }
    meet();
    if (mine > 0) {
        phase(0, sc, sc, T_{}, F_{}, [](auto) {});
        mask(0, sc);
    }
    meet();  // every wave has read K tile 0
    for (int t = 0; t + 1 < mine; ++t) iteration(t, T_{});
    if (mine > 0) iteration(mine - 1, F_{});
    if (mine < ntiles) meet();

    // Merge of the KS partial sweeps: every wave of a query block takes a
    // share of the output groups.  xs is read only after every wave wrote.
    l = halves_sum(l);
    const int64_t lidx = ((int64_t)b * a.H + hh) * a.Nq + qrow;
    // read by every wave of the query block before one of them overwrites it
    const float lse_prev = a.accum && qvalid ? a.lse[lidx] : -INFINITY;
    float* const xs = (float*)lds;
    float M = m, L = l, wgt[KS];
    if constexpr (KS > 1) {
        float* slot = xs + wave * C::XSLOT;
        slot[lane] = m;
        slot[64 + lane] = l;
#pragma unroll
        for (int db = 0; db < DBLK; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) slot[(2 + 16 * db + i) * 64 + lane] = o[db][i];
        if constexpr (C::TAIL)
#pragma unroll
            for (int i = 0; i < 8; ++i) slot[(2 + 4 * C::NG + i) * 64 + lane] = ot[i >> 2][i & 3];
        wait_vmem<0>();  // lse_prev has been read
        __syncthreads();
    }
    auto slot_of = [&](int k2) -> const float* { return xs + (k2 * QB + qb) * C::XSLOT; };
    // weights of the partial sweeps for the query of lane ql, and their sum
    auto weigh = [&](int ql, float (&w)[KS], float& Mq, float& Lq) {
        Mq = -INFINITY;
#pragma unroll
        for (int k2 = 0; k2 < KS; ++k2) Mq = fmaxf(Mq, slot_of(k2)[ql]);
        Lq = 0.f;
#pragma unroll
        for (int k2 = 0; k2 < KS; ++k2) {
            const float mk = slot_of(k2)[ql];
            w[k2] = mk == -INFINITY ? 0.f : exp_b2(mk - Mq);
            Lq = __builtin_fmaf(w[k2], slot_of(k2)[64 + ql], Lq);
        }
    };
    // (w_prev, w_new) of a query: L its weight sum, M its max; lse_out the merged LSE
    auto finish = [&](float Mq, float Lq, float prev, float& w_prev, float& w_new, float& lse_out) {
        const float lse_new = Lq > 0.f ? Mq + logf(Lq) : -INFINITY;
        // keys, but no finite score: 0/0
        const float inv = Lq > 0.f ? 1.f / Lq : (a.Nk > 0 ? NAN : 0.f);
        w_prev = 0.f;
        w_new = inv;
        lse_out = lse_new;
        if (prev != -INFINITY) {
            if (lse_new == -INFINITY) {
                w_prev = 1.f;
                w_new = a.Nk > 0 ? inv : 0.f;
                lse_out = prev;
            } else {
                const float Mx = fmaxf(prev, lse_new);
                const float e1 = expf(prev - Mx), e2 = expf(lse_new - Mx);
                w_prev = e1 / (e1 + e2);
                w_new = e2 / (e1 + e2) * inv;
                lse_out = Mx + logf(e1 + e2);
            }
        }
    };
    if constexpr (KS > 1) weigh(lane, wgt, M, L);
    float w_prev, w_new, lse_out;
    finish(M, L, lse_prev, w_prev, w_new, lse_out);
    float* const orow = a.out + ((int64_t)b * a.Nq + qrow) * rs + headoff;
    // rows 8g + 4hf .. +3 of the blocks are DBLK*4 consecutive dims: chunk q
    // of group g holds four of them, element f = 4q + e in block f % DBLK,
    // register 4g + f / DBLK
#pragma unroll
    for (int gq = 0; gq < C::NG; ++gq) {
        if (KS > 1 && gq % KS != kh) continue;
        const int g = gq / DBLK, q = gq % DBLK;
        f32x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int f = 4 * q + e, db = f % DBLK, i = 4 * g + f / DBLK;
            if constexpr (KS > 1) {
                y[e] = 0.f;
#pragma unroll
                for (int k2 = 0; k2 < KS; ++k2)
                    y[e] = __builtin_fmaf(wgt[k2], slot_of(k2)[(2 + 16 * db + i) * 64 + lane], y[e]);
            } else {
                y[e] = o[db][i];
            }
        }
        if (qvalid) store_row4(orow + DBLK * (8 * g + 4 * hf) + 4 * q, y * w_new, w_prev);
    }
    if constexpr (C::TAIL) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int ql = 16 * h + l16, qr = qt * C::BM + qb * 32 + ql;
            // the weights and state of this lane's tail query
            float wp, wn;
            f32x4 y = ot[h];
            if constexpr (KS > 1) {
                if (h % KS != kh) continue;
                float w2[KS], M2, L2, lo2;
                weigh(ql, w2, M2, L2);
                finish(M2, L2, __shfl(lse_prev, ql), wp, wn, lo2);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    y[e] = 0.f;
#pragma unroll
                    for (int k2 = 0; k2 < KS; ++k2)
                        y[e] = __builtin_fmaf(w2[k2], slot_of(k2)[(2 + 4 * C::NG + 4 * h + e) * 64 + lane], y[e]);
                }
            } else {
                wp = __shfl(w_prev, ql);
                wn = __shfl(w_new, ql);
            }
            if (grp < 2 && qr < a.Nq)
                store_row4(a.out + ((int64_t)b * a.Nq + qr) * rs + headoff + 64 + 4 * grp, y * wn, wp);
        }
    }
    if (a.lse && kh == 0 && hf == 0 && qvalid) a.lse[lidx] = lse_out;
}

template <int D, int QB, int KS, bool PATCH>
hipError_t launch(const AttnParams& p, hipStream_t s) {
    using C = FCfg<D, QB, KS>;
    F32Args a;
    a.q = (const float*)p.q;
    a.k = (const float*)p.k;
    a.v = (const float*)p.v;
    a.fk = (const float*)p.fresh_k;
    a.fv = (const float*)p.fresh_v;
    a.wk = (float*)p.wk;
    a.wv = (float*)p.wv;
    a.out = (float*)p.out;
    a.lse = p.lse;
    a.B = p.B;
    a.H = p.H;
    a.Nq = p.Nq;
    a.Nk = p.Nk;
    a.off0 = p.off0;
    a.len0 = p.len0;
    a.off1 = p.off1;
    a.len1 = p.len1;
    a.sa0 = p.len0 > 0 ? p.off0 / C::BN : 0;
    a.sn0 = p.len0 > 0 ? (p.off0 + p.len0 + C::BN - 1) / C::BN - a.sa0 : 0;
    a.sa1 = p.len1 > 0 ? p.off1 / C::BN : 0;
    a.sn1 = p.len1 > 0 ? (p.off1 + p.len1 + C::BN - 1) / C::BN - a.sa1 : 0;
    a.q_tiles = (p.Nq + C::BM - 1) / C::BM;
    a.scale = (float)(1.0 / sqrt((double)D));
    a.accum = p.accum;
    const int64_t blocks = (int64_t)a.q_tiles * p.H * p.B;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL((attn_f32_kernel<D, QB, KS, PATCH>), dim3((unsigned)blocks), dim3(C::THREADS), 0, s, a);
    return hipGetLastError();
}

// The key splits KS, by a model of the busiest CU in units of one 32-key tile
// of four waves (one per SIMD): its workgroups, each sweeping T / KS tiles
// plus a fixed part that grows with the exchange (0.5, 1, 1.3 and 1.5 tiles
// for KS = 1, 2, 4, 8).  Four waves alone on a CU run 10 % slower per tile
// than two such groups in turn; so do, by 20 %, the workgroups of KS = 4 at
// d = 128, whose LDS admits one per CU.  Measured, us for KS = 1 / 2 / 4 / 8:
//   2 x 16 heads of 72, 1024 queries, 1024 keys   101 / 94 / 100 / 119
//   24 heads of 64, 1000 queries, 1000 keys        79 /  75 /  62 /  70
//   24 heads of 64, 16 queries, 2500 keys         187 /  97 /  55 /  52
//   2 x 3 heads of 64, 40 queries, 1505 keys      115 /  60 /  34 /  33
//   24 heads of 128, 512 queries, 1024 keys       141 /  79 /  90
//   12 heads of 128, 256 queries, 2000 keys       270 / 143 /  83
template <int D, bool PATCH>
hipError_t dispatch(const AttnParams& p, hipStream_t s) {
    const int64_t bh = (int64_t)p.B * p.H;
    const int tiles = (p.Nk + kKT - 1) / kKT;
    const double fixed[4] = {0.5, 1.0, 1.3, 1.5};
    int ks = 1;
    double best = 0;
    for (int n = 0; n < (D > 96 ? 3 : 4); ++n) {
        const int k = 1 << n, qb = n < 2 ? 4 >> n : 1;
        const int64_t wgs = (p.Nq + 32 * qb - 1) / (32 * qb) * bh;
        const double quads = (double)((wgs + 255) / 256 * (qb * k / 4));
        double c = quads * ((tiles + k - 1) / k + fixed[n]);
        if (D > 96 && k == 4) c *= 1.2;
        else if (quads == 1) c *= 1.1;
        if (n == 0 || c < best) {
            best = c;
            ks = k;
        }
    }
    if constexpr (D <= 96)
        if (ks == 8) return launch<D, 1, 8, PATCH>(p, s);
    if (ks == 4) return launch<D, 1, 4, PATCH>(p, s);
    if (ks == 2) return launch<D, 2, 2, PATCH>(p, s);
    return launch<D, 4, 1, PATCH>(p, s);
}

}  // namespace

hipError_t launch_attn_f32(const AttnParams& p, hipStream_t s) {
    const bool patch = p.fresh_k != nullptr;
    switch (p.D) {
        case 64: return patch ? dispatch<64, true>(p, s) : dispatch<64, false>(p, s);
        case 72: return patch ? dispatch<72, true>(p, s) : dispatch<72, false>(p, s);
        case 128: return patch ? dispatch<128, true>(p, s) : dispatch<128, false>(p, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace xdit
