// pk_inst_gemm_tt.hip -- GEMM instances for op(A) = A^T, op(B) = B^T.
// Generated by gen_instances.py.
#include "pk_instance_common.hpp"

namespace pk {

const Config *configs_gemm_tt(int *count)
{
    static const Config kTable[] = {
        PK_GEMM(gemm_128x128x16_w2x2_tt_v44, 128, 128, 16, 2, 2, 1, 1, 4, 4, 1),
        PK_GEMM(gemm_64x64x16_w2x2_tt_v44, 64, 64, 16, 2, 2, 1, 1, 4, 4, 1),
        PK_GEMM(gemm_64x64x16_w2x2_tt_v11, 64, 64, 16, 2, 2, 1, 1, 1, 1, 1),
        PK_GEMM_DMA(gemm_256x256x32_w2x4_tt_v44_o2_dma2, 256, 256, 32, 2, 4, 2, 1, 1, 2),
        PK_GEMM_DMA(gemm_128x128x32_w2x4_tt_v44_o2_dma2, 128, 128, 32, 2, 4, 2, 1, 1, 2),
        PK_GEMM_DMA(gemm_64x64x32_w2x2_tt_v44_dma2, 64, 64, 32, 2, 2, 2, 1, 1, 1),
        PK_GEMM_DMA(gemm_64x64x16_w2x2_tt_v44_dma3, 64, 64, 16, 2, 2, 3, 1, 1, 1),
        PK_GEMM_DMA(gemm_128x32x32_w4x1_tt_v44_dma2, 128, 32, 32, 4, 1, 2, 1, 1, 1),
        PK_GEMM_DMA(gemm_128x96x32_w4x1_tt_v44_dma2, 128, 96, 32, 4, 1, 2, 1, 1, 1),
        PK_GEMM_DMA(gemm_128x64x32_w2x2_tt_v44_dma2, 128, 64, 32, 2, 2, 2, 1, 1, 1),
        PK_GEMM_DMA(gemm_32x64x32_w1x2_tt_v44_dma3, 32, 64, 32, 1, 2, 3, 1, 1, 1),
        PK_GEMM_DMA_KS(gemm_32x64x32_w1x2_k4_tt_v44_dma3, 32, 64, 32, 1, 2, 4, 3, 1, 1, 1),
        PK_GEMM_DMA_KS(gemm_64x64x32_w2x2_k2_tt_v44_dma3, 64, 64, 32, 2, 2, 2, 3, 1, 1, 1),
        PK_GEMM_DMA_KS(gemm_64x64x32_w2x2_k4_tt_v44_dma2, 64, 64, 32, 2, 2, 4, 2, 1, 1, 1),
        PK_GEMM_DMA_U(gemm_256x256x32_w2x4_tt_v11_o2_dma2, 256, 256, 32, 2, 4, 2, 1, 1, 2),
        PK_GEMM_DMA_U(gemm_128x128x32_w2x4_tt_v11_o2_dma2, 128, 128, 32, 2, 4, 2, 1, 1, 2),
        PK_GEMM_DMA_U(gemm_64x64x32_w2x2_tt_v11_dma2, 64, 64, 32, 2, 2, 2, 1, 1, 1),
        PK_GEMM_DMA_U(gemm_64x64x16_w2x2_tt_v11_dma3, 64, 64, 16, 2, 2, 3, 1, 1, 1),
        PK_GEMM_DMA_U(gemm_128x32x32_w4x1_tt_v11_dma2, 128, 32, 32, 4, 1, 2, 1, 1, 1),
        PK_GEMM_DMA_U(gemm_128x96x32_w4x1_tt_v11_dma2, 128, 96, 32, 4, 1, 2, 1, 1, 1),
        PK_GEMM_DMA_U(gemm_128x64x32_w2x2_tt_v11_dma2, 128, 64, 32, 2, 2, 2, 1, 1, 1),
        PK_GEMM_DMA_U(gemm_32x64x32_w1x2_tt_v11_dma3, 32, 64, 32, 1, 2, 3, 1, 1, 1),
        PK_GEMM_DMA_KS_U(gemm_32x64x32_w1x2_k4_tt_v11_dma3, 32, 64, 32, 1, 2, 4, 3, 1, 1, 1),
        PK_GEMM_DMA_KS_U(gemm_64x64x32_w2x2_k2_tt_v11_dma3, 64, 64, 32, 2, 2, 2, 3, 1, 1, 1),
        PK_GEMM_DMA_KS_U(gemm_64x64x32_w2x2_k4_tt_v11_dma2, 64, 64, 32, 2, 2, 4, 2, 1, 1, 1),
    };
    *count = (int)(sizeof(kTable) / sizeof(kTable[0]));
    return kTable;
}

}  // namespace pk
