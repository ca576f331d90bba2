// MFMA NT GEMM for the bfloat16 products of the CLEAR-MoE layer (gfx950):
//     C[m, n] = epi( sum_k A[arow(m), k] * B_seg(m)[n, k] )
// with the operands of GemmDesc (kernels.h).  The general kernel of gemm.hip
// takes float32 and the shapes outside gemm_bf16_supported (gemm_bf16.hip).
//
// What bounds it and why it looks like this (MI355X, about 2.05 GHz under
// load; the 50432-row products of the DeiT-Base layer):
//   * operands go HBM/L2 -> LDS by buffer loads whose per-lane offset never
//     changes and whose scalar offset steps along k, so the loop has no
//     vector address arithmetic (the general kernel spends about 45 vector
//     and 45 scalar instructions per stage and wave on it);
//   * a stage row is 128 bytes of k: whole cache lines.  64-byte rows issue
//     twice the L2 requests (the dense fc2 278 against 254 us with the tile of
//     that time);
//   * the fragments of the next k step are read while the current step's
//     MFMAs run, across the stage barrier too;
//   * the MFMAs read B's rows in a permuted order (gb_col_of_slot), so a lane
//     ends with 8 consecutive columns per half tile; the rows are rounded,
//     staged through LDS and stored as whole 64- or 128-byte row pieces, past
//     the L2 for large outputs: on the 320 x 256 tile, partial-line stores cost
//     fc1 + GELU 316 against 304 us, and z that is written back through the L2
//     another 20 us.
// In the dense FFN (kernel time, both libraries on one card): fc1 + GELU, 50432
// x 3072 x 768, 371 us with the general kernel, 287 here (two workgroups on a
// CU); fc2, 50432 x 768 x 3072, 294 and 229 (320 x 256); at 25216 rows 183 and
// 148, 166 and 110.
#pragma once

#include "kernels.h"

namespace clearmoe {

namespace {

constexpr int kGbRow = 128;                      // bytes of k per stage row
constexpr int kGbXcds = 8;                       // MI355X: 8 XCDs of 32 CUs
constexpr uint32_t kGbOob = 0x80000000u;         // an offset past every operand here
enum { kEpiPlain = 0, kEpiGelu = 1, kEpiScale = 2 };

typedef __attribute__((address_space(3))) uint32_t gb_lds_u32;
typedef int gb_i32x4 __attribute__((ext_vector_type(4)));

// Buffer descriptor of `bytes` bytes at p (uniform values): a load at an
// offset outside it returns zeros.
__device__ __forceinline__ gb_i32x4 gb_desc(const void* p, int64_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    gb_i32x4 d;
    d.x = __builtin_amdgcn_readfirstlane(static_cast<int>(a & 0xffffffffu));
    d.y = __builtin_amdgcn_readfirstlane(static_cast<int>((a >> 32) & 0xffffu));   // stride 0
    d.z = __builtin_amdgcn_readfirstlane(static_cast<int>(bytes));
    d.w = kRawWord3;
    return d;
}

// Descriptor of part 0, 1 or 2 (uniform), chosen word by word: an index into
// an array of descriptors would go through scratch memory.
__device__ __forceinline__ gb_i32x4 gb_pick(const gb_i32x4& d0, const gb_i32x4& d1, const gb_i32x4& d2, int part) {
    gb_i32x4 d;
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = __builtin_amdgcn_readfirstlane(part == 0 ? d0[i] : part == 1 ? d1[i] : d2[i]);
    return d;
}

// 16 bytes per lane, buffer -> LDS at m0 + 16 * lane.  Inline asm: the
// compiler does not count these loads, the pipeline's explicit waits do.
__device__ __forceinline__ void gb_dma16(const gb_i32x4& d, uint32_t voff, uint32_t soff, uint32_t m0) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(m0), "v"(voff), "s"(d), "s"(soff)
                 : "memory", "m0");
}

// Store of a finished row piece; nt: a streaming store past the L2.
__device__ __forceinline__ void gb_store(u32x4* p, const u32x4& v, bool nt) {
    if (nt) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// This wave's outstanding loads down to N, its LDS reads done, then the
// workgroup barrier.
template <int N>
__device__ __forceinline__ void gb_wait_barrier() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// LDS rows of SB bytes hold their 16-byte chunk c at slot c ^ gb_swz(row):
// 16 consecutive rows of one chunk hit 16 different 16-byte bank groups.
template <int SB>
__device__ __forceinline__ int gb_swz(int r) {
    constexpr int CPR = SB / 16, RW = 16 / CPR;
    return (r / RW) % CPR;
}

// Column (within 32) that MFMA row slot s reads.  With B as the MFMA's first
// operand a lane's result v is row slot 8 (v/4) + 4 (lane/32) + v%4, so this
// order makes it column 16 (v/8) + 8 (lane/32) + v%8: eight consecutive
// columns per half of v.  (16 lanes still read 16 neighbouring rows.)
__device__ __forceinline__ int gb_col_of_slot(int s) {
    return 16 * (s >> 4) + 8 * ((s >> 2) & 1) + 4 * ((s >> 3) & 1) + (s & 3);
}

__device__ __forceinline__ int gb_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}

// What a workgroup works on: rows [m_lo, m_lo + rows) of segment seg, column
// tile nt.
struct GbTile {
    int64_t m_lo;
    int rows, seg, nt;
};

// The tile of this workgroup (false: none, uniform over the workgroup).
template <int BM>
__device__ __forceinline__ bool gb_tile(const GemmDesc& g, int mtiles, int ntiles, int group, int lane,
                                        GbTile& t) {
    // XCD x = workgroup % 8 owns the row tiles x, x + 8, ... and takes them in
    // groups, column tile by column tile (shared A and B rows in its L2;
    // leading row tiles on every XCD); the last mtiles % 8 row tiles are
    // spread tile by tile, so that every XCD has its share
    const int xcd = blockIdx.x % kGbXcds, local = blockIdx.x / kGbXcds;
    const int m8 = mtiles / kGbXcds, full = m8 / group;
    int mt, nt;
    if (local < m8 * ntiles) {
        int mi;
        if (local < full * group * ntiles) {
            const int gi = local / (group * ntiles), r = local - gi * group * ntiles;
            mi = gi * group + r % group;
            nt = r / group;
        } else {
            const int r = local - full * group * ntiles, gm = m8 - full * group;
            mi = full * group + r % gm;
            nt = r / gm;
        }
        mt = mi * kGbXcds + xcd;
    } else {
        // the last mtiles % 8 row tiles, spread tile by tile over the XCDs
        const int r = (local - m8 * ntiles) * kGbXcds + xcd;
        mt = m8 * kGbXcds + r / ntiles;
        nt = r % ntiles;
        if (mt >= mtiles) return false;
    }
    int64_t m_lo, m_hi;
    int seg = 0;
    if (g.seg_offsets != nullptr && !g.seg_merge) {
        // lane s holds segment s (at most 64): a prefix sum of the segments'
        // row tiles and a ballot find this tile's segment.  Offsets are
        // clamped to [0, M]: bad ones cannot reach outside the buffers.
        const int M = static_cast<int>(g.M);
        int lo = lane < g.nseg ? g.seg_offsets[lane] : 0, hi = lane < g.nseg ? g.seg_offsets[lane + 1] : 0;
        lo = lo < 0 ? 0 : (lo > M ? M : lo);
        hi = hi < lo ? lo : (hi > M ? M : hi);
        const int n_t = (hi - lo + BM - 1) / BM;
        const int tend = gb_incl_scan(n_t);
        const uint64_t hit = __ballot(lane < g.nseg && mt < tend);
        if (hit == 0) return false;
        seg = __builtin_ctzll(hit);
        const int t0 = __builtin_amdgcn_readlane(tend - n_t, seg);
        m_lo = __builtin_amdgcn_readlane(lo, seg) + static_cast<int64_t>(mt - t0) * BM;
        m_hi = __builtin_amdgcn_readlane(hi, seg);
    } else {
        int64_t lo = 0, hi = g.M;
        if (g.seg_offsets != nullptr) {
            lo = __builtin_amdgcn_readfirstlane(g.seg_offsets[0]);
            hi = __builtin_amdgcn_readfirstlane(g.seg_offsets[g.nseg]);
            lo = lo < 0 ? 0 : (lo > g.M ? g.M : lo);
            hi = hi < lo ? lo : (hi > g.M ? g.M : hi);
        }
        m_lo = lo + static_cast<int64_t>(mt) * BM;
        m_hi = hi;
        if (m_lo >= hi) return false;
    }
    t.m_lo = m_lo;
    t.rows = static_cast<int>(m_hi - m_lo < BM ? m_hi - m_lo : BM);
    t.seg = seg;
    t.nt = nt;
    return true;
}

// The parts of B for segment seg.
struct GbParts {
    const bf16_bits *b0, *b1, *b2;
};
__device__ __forceinline__ GbParts gb_parts(const GemmDesc& g, int seg) {
    // parts 1 and 2 belong to the segment's expert or, for pair segments, to
    // its experts a and b
    int e1 = seg, e2 = seg;
    if (g.pair_E > 0) pair_experts(seg, g.pair_E, e1, e2);
    GbParts p;
    p.b0 = static_cast<const bf16_bits*>(g.B) + static_cast<int64_t>(seg) * g.b_seg_stride;
    p.b1 = static_cast<const bf16_bits*>(g.B1) + static_cast<int64_t>(e1) * g.b1_seg_stride;
    p.b2 = static_cast<const bf16_bits*>(g.B2) + static_cast<int64_t>(e2) * g.b2_seg_stride;
    return p;
}

// Byte offset (k = 0, chunk at element kc) of local row r of A; absent rows
// and negative gather indices (padding rows) read zeros.
__device__ __forceinline__ uint32_t gb_a_offset(const GemmDesc& g, int64_t m_lo, int rows, int r, int kc) {
    uint32_t src = static_cast<uint32_t>(r);
    bool ok = r < rows;
    if (g.a_rows != nullptr) {
        const int32_t s = ok ? g.a_rows[m_lo + r] : -1;
        ok = s >= 0;
        src = static_cast<uint32_t>(g.a_div == 1 ? s : s / g.a_div);
    }
    return ok ? (src * static_cast<uint32_t>(g.lda) + static_cast<uint32_t>(kc)) * 2u : kGbOob;
}
__device__ __forceinline__ gb_i32x4 gb_a_desc(const GemmDesc& g, int64_t m_lo, int rows) {
    const bf16_bits* A = static_cast<const bf16_bits*>(g.A);
    return g.a_rows == nullptr ? gb_desc(A + m_lo * g.lda, ((static_cast<int64_t>(rows) - 1) * g.lda + g.K) * 2)
                               : gb_desc(A, g.a_nrows * g.lda * 2);
}

// Descriptor and byte offset of column n of B split along n.  ng, the first
// column of the load's eight, picks the part for every lane alike (parts
// start at multiples of 8 columns).
__device__ __forceinline__ uint32_t gb_b_offset(const GemmDesc& g, const GbParts& p, int ng, int n, int kc,
                                                gb_i32x4& d) {
    const GemmBPart b = gemm_b_part(g.N, g.n_split, g.n_split2, ng);
    const bf16_bits* base = b.part == 0 ? p.b0 : b.part == 1 ? p.b1 : p.b2;
    const int64_t ld = b.part == 0 ? g.ldb : b.part == 1 ? g.ldb1 : g.ldb2;
    d = gb_desc(base, static_cast<int64_t>(b.n1 - b.n0) * ld * 2);
    return n < b.n1 ? (static_cast<uint32_t>(n - b.n0) * static_cast<uint32_t>(ld) + static_cast<uint32_t>(kc)) * 2u
                    : kGbOob;
}

template <int TM, int TN>
__device__ __forceinline__ void gb_zero(f32x16 (&acc)[TM][TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
}

// Bias of column nw + lane (nw: the wave's first column; 0 past N or without a
// bias), loaded before the k loop and added after it: a register a lane in
// between.  An accumulator that starts at the bias rounds every partial sum
// at the bias's magnitude, and takes four times as many loads (1576 tokens,
// top-1, D = 768: the layer's three products 5 us more).
__device__ __forceinline__ float gb_bias(const GemmDesc& g, int nw, int lane) {
    const __amdgpu_buffer_rsrc_t rb = raw_rsrc(g.bias, g.bias != nullptr ? static_cast<int64_t>(g.N) * 4 : 0);
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rb, (nw + lane) * 4, 0, 0));
}

// Epilogue of one wave: local rows rw .. rw + 32 TM, columns nw .. nw + 32 TN.
// Lane l holds row .. + i * 32 + l % 32 and, per half h of a tile's 16
// values, 8 consecutive columns; N and ldc are multiples of 8, so a group is
// all in or all out.  bfloat16 rows go through wb, 32 rows of this wave's own
// LDS (16-byte chunks swizzled by the row), and leave as whole row pieces.
// bias: gb_bias of this lane, handed to the lanes that hold its column through
// the same LDS.
template <int TM, int TN, int EPI>
__device__ __forceinline__ void gb_epilogue(const GemmDesc& g, const GbTile& t, int rw, int nw, int lane,
                                            unsigned char* wb, bool nt, float bias, f32x16 (&acc)[TM][TN]) {
    const int lrow = lane & 31, lh = lane >> 5;
    static_assert(TN <= 2, "a lane for every column of the wave");
    if constexpr (EPI != kEpiScale) {                             // a scaled product has no bias
        reinterpret_cast<float*>(wb)[lane] = bias;
        __builtin_amdgcn_wave_barrier();
        f32x4 b4[TN][4];
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int h = 0; h < 4; ++h)
                b4[j][h] = *reinterpret_cast<const f32x4*>(wb + 4 * (j * 32 + 16 * (h >> 1) + 8 * lh + 4 * (h & 1)));
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] += b4[j][v >> 2][v & 3];
    }
    constexpr int RB = TN * 64, CH = RB / 16, RPI = 64 / CH;      // row bytes, chunks, rows per store
    static_assert(64 % CH == 0 && 32 % RPI == 0, "whole rows per store");
    if (EPI == kEpiPlain && g.c_f32) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int rl = rw + i * 32 + lrow;
            if (rl >= t.rows) continue;
            int64_t cm = t.m_lo + rl;
            if (g.c_rows != nullptr) {
                const int32_t cr = g.c_rows[cm];
                if (cr < 0) continue;                   // a padding row is not stored
                cm = g.c_div == 1 ? cr : cr / g.c_div;
            }
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int n = nw + j * 32 + 16 * h + 8 * lh;
                    if (n >= g.N) continue;
                    float* c = static_cast<float*>(g.C) + cm * g.ldc + n;
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        *reinterpret_cast<float4*>(c + 4 * q) =
                            make_float4(acc[i][j][8 * h + 4 * q], acc[i][j][8 * h + 4 * q + 1],
                                        acc[i][j][8 * h + 4 * q + 2], acc[i][j][8 * h + 4 * q + 3]);
                }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        float rs = 1.0f, rs1 = 1.0f;
        if constexpr (EPI == kEpiScale) {
            const int rl = rw + i * 32 + lrow;
            const int32_t sr = rl < t.rows ? g.scale_rows[t.m_lo + rl] : -1;
            rs = sr >= 0 ? g.row_scale[sr] : 0.0f;
            rs1 = g.row_scale2 == nullptr ? rs : (sr >= 0 ? g.row_scale2[sr] : 0.0f);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int n = nw + j * 32 + 16 * h + 8 * lh;
                float v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = acc[i][j][8 * h + q];
                if constexpr (EPI == kEpiScale) {
                    const float sc = n >= g.scale_col0 ? (n >= g.scale_col1 ? rs1 : rs) : 1.0f;
#pragma unroll
                    for (int q = 0; q < 8; ++q) v[q] *= sc;
                }
                if constexpr (EPI == kEpiGelu) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) v[q] = gelu_erf(v[q]);
                }
                u32x4 w;
                w.x = pack2_bf16(v[0], v[1]);
                w.y = pack2_bf16(v[2], v[3]);
                w.z = pack2_bf16(v[4], v[5]);
                w.w = pack2_bf16(v[6], v[7]);
                const int ch = j * 4 + 2 * h + lh;
                *reinterpret_cast<u32x4*>(wb + lrow * RB + ((ch ^ (lrow % CH)) << 4)) = w;
            }
        // one wave's LDS accesses complete in order: only the compiler has to
        // keep them in place
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < 32 / RPI; ++it) {
            const int rr = it * RPI + lane / CH, ch = lane % CH;
            const u32x4 w = *reinterpret_cast<const u32x4*>(wb + rr * RB + ((ch ^ (rr % CH)) << 4));
            const int rl = rw + i * 32 + rr, n = nw + ch * 8;
            if (rl < t.rows && n < g.N) {
                int64_t cm = t.m_lo + rl;
                if (g.c_rows != nullptr) {
                    const int32_t cr = g.c_rows[cm];
                    cm = cr < 0 ? -1 : (g.c_div == 1 ? cr : cr / g.c_div);
                }
                if (cm < 0) continue;                   // a padding row is not stored
                u32x4 o = w;
                if (EPI == kEpiPlain && g.res != nullptr)
                    o = add8_bf16(o, *reinterpret_cast<const u32x4*>(static_cast<const bf16_bits*>(g.res) +
                                                                     cm * g.ldr + n));
                gb_store(reinterpret_cast<u32x4*>(static_cast<bf16_bits*>(g.C) + cm * g.ldc + n), o, nt);
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// WM x WN waves, each TM x TN MFMA tiles of 32 x 32; NS stages of 64 k in
// LDS; OCC waves per SIMD.  KS3: B changes part along k (see GemmDesc): each
// part has whole stages of its own, the last one filled up with zeros.  Else
// along n.
template <int WM, int WN, int TM, int TN, int NS, int OCC, int EPI, bool KS3>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(OCC, OCC)))
void k_gemm_bf16(GemmDesc g, int mtiles, int ntiles, int group, int nt_store) {
    constexpr int NW = WM * WN, SB = kGbRow;
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    constexpr int CPR = SB / 16, RPL = 64 / CPR;        // chunks per row, rows per load
    constexpr int KS = SB / 32, BK = SB / 2;            // 16-wide k steps per stage, k per stage
    constexpr int AL = BM / (RPL * NW), BL = BN / (RPL * NW), LPS = AL + BL;
    static_assert(BM % (RPL * NW) == 0 && BN % (RPL * NW) == 0, "whole loads per wave");
    static_assert(NS >= 2 && NS <= 3 && LPS * (NS - 1) < 64, "pipeline");
    constexpr int STAGE_A = BM * SB, STAGE = (BM + BN) * SB;
    static_assert(NS * STAGE >= NW * 32 * TN * 64, "the epilogue's rows fit the stages");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[NS * STAGE];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int lrow = lane & 31, lh = lane >> 5;

    GbTile t;
    if (!gb_tile<BM>(g, mtiles, ntiles, group, lane, t)) return;
    const int n0 = t.nt * BN;
    const GbParts bp = gb_parts(g, t.seg);

    // ---- per-lane byte offsets of the loads at k = 0: load i brings 8 rows
    const int lr = lane / CPR, cp = lane % CPR;
    const gb_i32x4 da = gb_a_desc(g, t.m_lo, t.rows);
    uint32_t va[AL], vb[BL], vb1[KS3 ? BL : 1];
    // first k of the lane's chunk in LDS row r
    auto chunk_k = [&](int r) { return 8 * (cp ^ gb_swz<SB>(r)); };
#pragma unroll
    for (int i = 0; i < AL; ++i) {
        const int r = (wave * AL + i) * RPL + lr;
        va[i] = gb_a_offset(g, t.m_lo, t.rows, r, chunk_k(r));
    }
    gb_i32x4 db[KS3 ? 3 : BL];
    if constexpr (KS3) {
        db[0] = gb_desc(bp.b0, static_cast<int64_t>(g.N) * g.ldb * 2);
        db[1] = gb_desc(bp.b1, static_cast<int64_t>(g.N) * g.ldb1 * 2);
        db[2] = gb_desc(bp.b2, static_cast<int64_t>(g.N) * g.ldb2 * 2);
    }
#pragma unroll
    for (int i = 0; i < BL; ++i) {
        const int r = (wave * BL + i) * RPL + lr;
        const int n = n0 + r;
        if constexpr (KS3) {
            const uint32_t kc = static_cast<uint32_t>(chunk_k(r));
            vb[i] = n < g.N ? (static_cast<uint32_t>(n) * static_cast<uint32_t>(g.ldb) + kc) * 2u : kGbOob;
            vb1[i] = n < g.N ? (static_cast<uint32_t>(n) * static_cast<uint32_t>(g.ldb1) + kc) * 2u : kGbOob;
        } else {
            vb[i] = gb_b_offset(g, bp, n0 + (wave * BL + i) * RPL, n, chunk_k(r), db[i]);
        }
    }

    // stages: all of K, or with KS3 those of the parts one after the other
    const int k1 = g.k_split < g.K ? g.k_split : g.K, k2 = g.k_split2 < g.K ? g.k_split2 : g.K;
    const int s1 = (k1 + BK - 1) / BK, s2 = s1 + (k2 - k1 + BK - 1) / BK;
    const int nk = KS3 ? s2 + (g.K - k2 + BK - 1) / BK : (g.K + BK - 1) / BK;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((gb_lds_u32*)smem)));

    // load i of stage kt into LDS buffer b
    auto dma = [&](int kt, int b, int i) {
        // first k of the stage in A and in the part of B, and k left there
        int ka = kt * BK, kb = ka, left = g.K - ka;
        int part = 0;
        if constexpr (KS3) {
            left = k1 - ka;
            if (kt >= s2) {
                kb = (kt - s2) * BK; ka = k2 + kb; left = g.K - ka; part = 2;
            } else if (kt >= s1) {
                kb = (kt - s1) * BK; ka = k1 + kb; left = k2 - ka; part = 1;
            }
        }
        const bool cut = left < BK;                     // uniform: chunks past the end read zeros
        if (i < AL) {
            const int r = (wave * AL + i) * RPL + lr;
            uint32_t v = va[i < AL ? i : 0];
            if (cut) v = chunk_k(r) < left ? v : kGbOob;
            gb_dma16(da, v, __builtin_amdgcn_readfirstlane(ka * 2),
                     __builtin_amdgcn_readfirstlane(lds0 + b * STAGE + (wave * AL + i) * 1024));
        } else {
            const int q = i - AL < BL && i >= AL ? i - AL : 0;
            const int r = (wave * BL + q) * RPL + lr;
            uint32_t v = vb[q];
            gb_i32x4 d;
            if constexpr (KS3) {
                v = part > 0 ? vb1[q] : v;
                d = gb_pick(db[0], db[1], db[2], part);
            } else {
                d = db[q];
            }
            if (cut) v = chunk_k(r) < left ? v : kGbOob;
            gb_dma16(d, v, __builtin_amdgcn_readfirstlane(kb * 2),
                     __builtin_amdgcn_readfirstlane(lds0 + b * STAGE + STAGE_A + (wave * BL + q) * 1024));
        }
    };
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s < nk) {
#pragma unroll
            for (int i = 0; i < LPS; ++i) dma(s, s, i);
        }

    const float bias = gb_bias(g, n0 + wn * TN * 32, lane);
    f32x16 acc[TM][TN];
    gb_zero(acc);

    // byte offsets of this lane's operand chunks of k step s within a stage
    const int bcol = gb_col_of_slot(lrow);
    uint32_t oa[KS], ob[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        oa[s] = static_cast<uint32_t>((wm * TM * 32 + lrow) * SB + (((2 * s + lh) ^ gb_swz<SB>(lrow)) << 4));
        ob[s] = static_cast<uint32_t>(STAGE_A + (wn * TN * 32 + bcol) * SB +
                                      (((2 * s + lh) ^ gb_swz<SB>(bcol)) << 4));
    }
    u32x4 fa[2][TM], fb[2][TN];
    auto read = [&](int b, int s, int p) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
            fb[p][j] = *reinterpret_cast<const u32x4*>(smem + b * STAGE + ob[s] + j * 32 * SB);
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[p][i] = *reinterpret_cast<const u32x4*>(smem + b * STAGE + oa[s] + i * 32 * SB);
    };

    // stage 0 has landed for every wave (the later ones may be in flight)
    if (NS >= 3 && nk >= 3) gb_wait_barrier<(NS >= 3 ? 2 * LPS : 0)>();
    else if (nk >= 2) gb_wait_barrier<LPS>();
    else gb_wait_barrier<0>();
    read(0, 0, 0);

    for (int k0 = 0; k0 < nk; k0 += NS) {
#pragma unroll
        for (int b = 0; b < NS; ++b) {
            const int kt = k0 + b;
            if (kt >= nk) break;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const int p = s & 1;
                if (s < KS - 1) {
                    read(b, s + 1, p ^ 1);
                } else if (kt + 1 < nk) {
                    // stage kt + 1 has landed for every wave, and every wave
                    // is done reading stage kt's buffer, which takes kt + NS
                    if (NS >= 3 && kt + 2 < nk) gb_wait_barrier<(NS >= 3 ? LPS : 0)>();
                    else gb_wait_barrier<0>();
                    read((b + 1) % NS, 0, p ^ 1);
                    if (kt + NS < nk) {
#pragma unroll
                        for (int i = 0; i < LPS; ++i) dma(kt + NS, b, i);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            __builtin_bit_cast(bf16x8, fb[p][j]), __builtin_bit_cast(bf16x8, fa[p][i]),
                            acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    gb_wait_barrier<0>();                       // the stage buffers are free
    gb_epilogue<TM, TN, EPI>(g, t, wm * TM * 32, n0 + wn * TN * 32, lane, smem + wave * (32 * TN * 64),
                             nt_store != 0, bias, acc);
}

// 256 x 256 tile over eight waves (2 x 4, each 128 x 64), two stages of 64 k:
// the variant for long k.  A stage is consumed in two phases, the upper and
// the lower 64 rows of each wave's A, and a wave holds a whole phase's
// fragments in registers: the LDS of B and of A's upper half is free as soon
// as phase 0 starts, that of the lower half when phase 1 does, so the loads of
// stage kt + 2 are issued one and a half to two stages before they are read
// (one with the kernel above: 902 us for 65536 x 1024 x 8192 on a 256 x 256
// tile of it).  Against the 320 x 256 tile: 65536 x 1024 x 8192 827 and 1066
// us (1330 TFLOP/s), 50432 x 384 x 1536 80 and 103, 50432 x 768 x 3072 234 and
// 232, 25216 x 768 x 3072 139 and 110: what the tiles leave of the last round
// decides.
template <int EPI>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_bf16_long(GemmDesc g, int mtiles, int ntiles, int group, int nt_store) {
    constexpr int SB = kGbRow, BM = 256, BN = 256, CPR = 8, BK = 64, TM = 4, TN = 2;
    constexpr int BUF = BM * SB;                        // buffers A0 A1 B0 B1
    __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * BUF];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / 4, wn = wave % 4;
    const int lrow = lane & 31, lh = lane >> 5;

    GbTile t;
    if (!gb_tile<BM>(g, mtiles, ntiles, group, lane, t)) return;
    const int n0 = t.nt * BN;
    const GbParts bp = gb_parts(g, t.seg);

    const int lr = lane / CPR, cp = lane % CPR;
    const gb_i32x4 da = gb_a_desc(g, t.m_lo, t.rows);
    // first k of the lane's chunk in an even load's 8 rows; odd: ^ 32
    const int kc0 = 8 * (cp ^ (lr >> 1));
    uint32_t va[4], vb[4];
    int ra[4];
    gb_i32x4 db[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // loads 0, 1: rows [0, 64) of each wave row's 128; 2, 3: [64, 128)
        const int q = wave * 2 + (i & 1);
        const int r8 = (q < 8 ? q : q + 8) + (i >= 2 ? 8 : 0);
        ra[i] = r8 * 1024;
        va[i] = gb_a_offset(g, t.m_lo, t.rows, r8 * 8 + lr, kc0 ^ (32 * (i & 1)));
        const int r = (wave * 4 + i) * 8 + lr;
        const int n = n0 + r;
        vb[i] = gb_b_offset(g, bp, n0 + (wave * 4 + i) * 8, n, kc0 ^ (32 * (i & 1)), db[i]);
    }
    const int nk = (g.K + BK - 1) / BK, K = g.K;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((gb_lds_u32*)smem)));
    // stages past the last are issued too (zeros, no memory traffic), so that
    // every wait below counts the same
    auto masked = [&](uint32_t v, int kt, int i) {
        if ((kt + 1) * BK > K) v = kt * BK + (kc0 ^ (32 * (i & 1))) < K ? v : kGbOob;
        return v;
    };
    auto dma_a = [&](int kt, int b, int i) {
        gb_dma16(da, masked(va[i], kt, i), __builtin_amdgcn_readfirstlane((kt < nk ? kt : 0) * BK * 2),
                 __builtin_amdgcn_readfirstlane(lds0 + b * BUF + ra[i]));
    };
    auto dma_b = [&](int kt, int b, int i) {
        gb_dma16(db[i], masked(vb[i], kt, i), __builtin_amdgcn_readfirstlane((kt < nk ? kt : 0) * BK * 2),
                 __builtin_amdgcn_readfirstlane(lds0 + (2 + b) * BUF + (wave * 4 + i) * 1024));
    };
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
        for (int i = 0; i < 4; ++i) dma_b(s, s, i);
#pragma unroll
        for (int i = 0; i < 4; ++i) dma_a(s, s, i);
    }
    const float bias = gb_bias(g, n0 + wn * TN * 32, lane);
    f32x16 acc[TM][TN];
    gb_zero(acc);

    const int bcol = gb_col_of_slot(lrow);
    uint32_t oa[4], ob[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        oa[s] = static_cast<uint32_t>((wm * 128 + lrow) * SB + (((2 * s + lh) ^ gb_swz<SB>(lrow)) << 4));
        ob[s] = static_cast<uint32_t>(2 * BUF + (wn * 64 + bcol) * SB + (((2 * s + lh) ^ gb_swz<SB>(bcol)) << 4));
    }
    u32x4 fu[2][4], fl[2][4], fb[2][4];          // A upper, A lower, B: [tile][k step]
    auto rd_a = [&](int b, int i, int s) {
        return *reinterpret_cast<const u32x4*>(smem + oa[s] + b * BUF + i * 32 * SB);
    };
    auto rd_b = [&](int b, int j, int s) {
        return *reinterpret_cast<const u32x4*>(smem + ob[s] + b * BUF + j * 32 * SB);
    };
    auto mm = [&](f32x16& c, const u32x4& a, const u32x4& b) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, b), __builtin_bit_cast(bf16x8, a),
                                                    c, 0, 0, 0);
    };
    gb_wait_barrier<8>();                        // stage 0 has landed
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        fb[0][s] = rd_b(0, 0, s);
        fb[1][s] = rd_b(0, 1, s);
        fu[0][s] = rd_a(0, 0, s);
        fu[1][s] = rd_a(0, 1, s);
    }
    for (int k0 = 0; k0 < nk; k0 += 2) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int kt = k0 + b;
            if (kt >= nk) break;
            // phase 0: B and A's upper rows of stage kt are in every wave's
            // registers; A's lower rows have landed (after them: 6 loads of
            // stage kt + 1's B and upper A, 2 of its lower A)
            gb_wait_barrier<8>();
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                fl[0][s] = rd_a(b, 2, s);
                fl[1][s] = rd_a(b, 3, s);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    mm(acc[0][j], fu[0][s], fb[j][s]);
                    mm(acc[1][j], fu[1][s], fb[j][s]);
                    if (s < 2) dma_b(kt + 2, b, 2 * s + j);
                    if (s == 2) dma_a(kt + 2, b, j);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // phase 1: stage kt + 1's B and upper A have landed (after them:
            // 2 loads of its lower A, 6 of stage kt + 2); stage kt's lower A
            // is in registers
            gb_wait_barrier<8>();
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                fu[0][s] = rd_a(b ^ 1, 0, s);
                fu[1][s] = rd_a(b ^ 1, 1, s);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    mm(acc[2][j], fl[0][s], fb[j][s]);
                    mm(acc[3][j], fl[1][s], fb[j][s]);
                    fb[j][s] = rd_b(b ^ 1, j, s);
                    if (s == 0) dma_a(kt + 2, b, 2 + j);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }
    gb_wait_barrier<0>();                        // the stage buffers are free
    gb_epilogue<TM, TN, EPI>(g, t, wm * TM * 32, n0 + wn * TN * 32, lane, smem + wave * (32 * TN * 64),
                             nt_store != 0, bias, acc);
}

// fc1 + GELU over many rows: 256 x 128 tile over four waves (2 x 2, each 128 x
// 64), two workgroups on a CU.  A tile's GELUs take about as many vector cycles
// as its k loop takes matrix cycles at K = 768 (80 each, four of a wave's
// instructions being quarter rate), and its rows a third of the time in
// stores; a single workgroup of the tiles above has nothing to run beside
// them, here one workgroup's epilogue runs beside the other's MFMAs.  80 KB of
// LDS each: A has two stage buffers, B one, which is free as soon as its
// fragments (a whole stage's, read first) are in registers.
// Against the better of the tiles above, in the dense FFN: 50432 x 3072 x 768
// 322 and 288 us, 50432 x 1536 x 384 115 and 100, 25216 x 3072 x 768 160 and
// 150.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_gemm_bf16_duo(GemmDesc g, int mtiles, int ntiles, int group, int nt_store) {
    constexpr int SB = kGbRow, BM = 256, BN = 128, CPR = 8, BK = 64, TM = 4, TN = 2, AL = 8, BL = 4;
    constexpr int ABUF = BM * SB, BOFF = 2 * ABUF;      // buffers A0 A1 B
    __shared__ __attribute__((aligned(1024))) unsigned char smem[BOFF + BN * SB];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = lane & 31, lh = lane >> 5;

    GbTile t;
    if (!gb_tile<BM>(g, mtiles, ntiles, group, lane, t)) return;
    const int n0 = t.nt * BN;
    const GbParts bp = gb_parts(g, t.seg);

    const int lr = lane / CPR, cp = lane % CPR;
    const gb_i32x4 da = gb_a_desc(g, t.m_lo, t.rows);
    // first k of the lane's chunk in an even load's 8 rows; odd: ^ 32
    const int kc0 = 8 * (cp ^ (lr >> 1));
    uint32_t va[AL], vb[BL];
    gb_i32x4 db[BL];
#pragma unroll
    for (int i = 0; i < AL; ++i)
        va[i] = gb_a_offset(g, t.m_lo, t.rows, (wave * AL + i) * 8 + lr, kc0 ^ (32 * (i & 1)));
#pragma unroll
    for (int i = 0; i < BL; ++i)
        vb[i] = gb_b_offset(g, bp, n0 + (wave * BL + i) * 8, n0 + (wave * BL + i) * 8 + lr, kc0 ^ (32 * (i & 1)),
                            db[i]);
    const int nk = (g.K + BK - 1) / BK, K = g.K;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((gb_lds_u32*)smem)));
    auto masked = [&](uint32_t v, int kt, int i) {
        if ((kt + 1) * BK > K) v = kt * BK + (kc0 ^ (32 * (i & 1))) < K ? v : kGbOob;
        return v;
    };
    auto dma_a = [&](int kt, int b) {
#pragma unroll
        for (int i = 0; i < AL; ++i)
            gb_dma16(da, masked(va[i], kt, i), __builtin_amdgcn_readfirstlane(kt * BK * 2),
                     __builtin_amdgcn_readfirstlane(lds0 + b * ABUF + (wave * AL + i) * 1024));
    };
    auto dma_b = [&](int kt) {
#pragma unroll
        for (int i = 0; i < BL; ++i)
            gb_dma16(db[i], masked(vb[i], kt, i), __builtin_amdgcn_readfirstlane(kt * BK * 2),
                     __builtin_amdgcn_readfirstlane(lds0 + BOFF + (wave * BL + i) * 1024));
    };
    dma_a(0, 0);
    dma_b(0);
    const float bias = gb_bias(g, n0 + wn * TN * 32, lane);
    f32x16 acc[TM][TN];
    gb_zero(acc);

    const int bcol = gb_col_of_slot(lrow);
    uint32_t oa[4], ob[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        oa[s] = static_cast<uint32_t>((wm * 128 + lrow) * SB + (((2 * s + lh) ^ gb_swz<SB>(lrow)) << 4));
        ob[s] = static_cast<uint32_t>(BOFF + (wn * 64 + bcol) * SB + (((2 * s + lh) ^ gb_swz<SB>(bcol)) << 4));
    }
    u32x4 fa[2][TM], fb[4][TN];
    auto read_a = [&](int b, int s) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
            fa[s & 1][i] = *reinterpret_cast<const u32x4*>(smem + oa[s] + b * ABUF + i * 32 * SB);
    };
    auto mm = [&](int s) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, fb[s][j]), __builtin_bit_cast(bf16x8, fa[s & 1][i]),
                    acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int k0 = 0; k0 < nk; k0 += 2) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int kt = k0 + b;
            if (kt >= nk) break;
            // stage kt has landed for every wave, and every wave is done
            // reading the other A buffer
            gb_wait_barrier<0>();
            if (kt + 1 < nk) dma_a(kt + 1, b ^ 1);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                fb[0][j] = *reinterpret_cast<const u32x4*>(smem + ob[0] + j * 32 * SB);
            read_a(b, 0);
#pragma unroll
            for (int s = 1; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    fb[s][j] = *reinterpret_cast<const u32x4*>(smem + ob[s] + j * 32 * SB);
            read_a(b, 1);
            mm(0);
            if (kt + 1 < nk) {
                // every wave has read this stage's B
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                dma_b(kt + 1);
            }
            read_a(b, 2);
            mm(1);
            read_a(b, 3);
            mm(2);
            mm(3);
        }
    }
    gb_wait_barrier<0>();                        // the stage buffers are free
    gb_epilogue<TM, TN, kEpiGelu>(g, t, wm * TM * 32, n0 + wn * TN * 32, lane, smem + wave * (32 * TN * 64),
                             nt_store != 0, bias, acc);
}

template <int BM, int BN>
bool gb_grid(const GemmDesc& g, int64_t& mt, int64_t& nt) {
    mt = (g.M + BM - 1) / BM;
    if (g.seg_offsets != nullptr && !g.seg_merge) mt += g.nseg;
    nt = (g.N + BN - 1) / BN;
    return mt * nt > 0;
}

// Outputs of kGbStreamBytes or more are written past the L2.
constexpr int64_t kGbStreamBytes = 16 << 20;
inline int gb_stream(const GemmDesc& g) {
    return !g.c_f32 && g.M * static_cast<int64_t>(g.N) * 2 >= kGbStreamBytes ? 1 : 0;
}

template <int WM, int WN, int TM, int TN, int NS, int OCC, int EPI, bool KS3>
hipError_t gemm_bf16_cfg(const GemmDesc& g, hipStream_t st) {
    int64_t mt, nt;
    if (!gb_grid<WM * TM * 32, WN * TN * 32>(g, mt, nt)) return hipSuccess;
    const int64_t grid = (mt * nt + kGbXcds - 1) / kGbXcds * kGbXcds;
    launch_kernel(k_gemm_bf16<WM, WN, TM, TN, NS, OCC, EPI, KS3>, dim3(static_cast<unsigned>(grid)),
                  64 * WM * WN, 0, st, g, static_cast<int>(mt), static_cast<int>(nt), 4, gb_stream(g));
    return hipGetLastError();
}

template <int EPI>
hipError_t gemm_bf16_long(const GemmDesc& g, hipStream_t st) {
    int64_t mt, nt;
    if (!gb_grid<256, 256>(g, mt, nt)) return hipSuccess;
    const int64_t grid = (mt * nt + kGbXcds - 1) / kGbXcds * kGbXcds;
    launch_kernel(k_gemm_bf16_long<EPI>, dim3(static_cast<unsigned>(grid)), 512, 0, st, g,
                  static_cast<int>(mt), static_cast<int>(nt), 4, gb_stream(g));
    return hipGetLastError();
}

inline hipError_t gemm_bf16_duo(const GemmDesc& g, hipStream_t st) {
    int64_t mt, nt;
    if (!gb_grid<256, 128>(g, mt, nt)) return hipSuccess;
    const int64_t grid = (mt * nt + kGbXcds - 1) / kGbXcds * kGbXcds;
    launch_kernel(k_gemm_bf16_duo, dim3(static_cast<unsigned>(grid)), 256, 0, st, g,
                  static_cast<int>(mt), static_cast<int>(nt), 4, gb_stream(g));
    return hipGetLastError();
}

}  // namespace

}  // namespace clearmoe
